"""Simplification and edge listing around vertices of many faces: where a ring
leaves the vertex's slots, is sorted by a wave, by a workgroup in LDS and in
global memory, and where the room for long rings runs out.  Bit for bit the FP64
oracle's."""
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from synth import meshes as M  # noqa: E402


def poles(k, seed, caps=2, rows=2):
    """Rings of k vertices between poles of k faces each (an open end is a boundary)."""
    rng = np.random.default_rng(seed)
    th = 2 * np.pi * np.arange(k) / k
    V = [[0, 0, 1.2]]
    for r in range(rows):
        V += np.stack([np.cos(th + 0.3 * r), np.sin(th + 0.3 * r), np.full(k, 0.4 - 0.8 * r / max(1, rows - 1))], 1).tolist()
    V += [[0, 0, -1.2]]
    at = lambda r, i: 1 + r * k + i % k  # noqa: E731
    F = [[0, at(0, i), at(0, i + 1)] for i in range(k)]
    for r in range(rows - 1):
        for i in range(k):
            F += [[at(r, i), at(r + 1, i), at(r, i + 1)], [at(r, i + 1), at(r + 1, i), at(r + 1, i + 1)]]
    if caps > 1:
        F += [[len(V) - 1, at(rows - 1, i + 1), at(rows - 1, i)] for i in range(k)]
    V = np.array(V) + rng.normal(size=(len(V), 3)) * 0.3 / k
    return V, np.array(F)


def kis(V, F, times):
    """Each face split at its centre: doubles every old vertex's faces."""
    for _ in range(times):
        n = len(V) + np.arange(len(F))
        C = V[F].mean(1)
        V = np.concatenate([V, C / np.linalg.norm(C, axis=1, keepdims=True)])
        F = np.concatenate([np.stack([F[:, i], F[:, (i + 1) % 3], n], 1) for i in range(3)])
    return V, F


def two_fans(k, seed):
    """Two fans of k faces that share their tip alone, and a third inside out."""
    rng = np.random.default_rng(seed)
    V, F = [np.zeros(3)], []
    for f in range(3):
        b = len(V)
        th = np.linspace(0, 3, k + 1)
        V += list(np.stack([np.cos(th), np.sin(th), np.full(k + 1, f - 1.0)], 1) + rng.normal(size=(k + 1, 3)) * 0.02)
        F += [[0, b + i, b + i + 1] if f < 2 else [b + i, 0, b + i + 1] for i in range(k)]
    return np.array(V), np.array(F)


def edges_of_one_face(n_v, seed):
    """Triangles on few vertices, no two with an edge in common: the most ring
    entries per face and per vertex."""
    rng = np.random.default_rng(seed)
    used, F = np.zeros((n_v, n_v), bool), []
    for _ in range(60 * n_v * n_v):
        a, b, c = rng.choice(n_v, 3, replace=False)
        if not (used[a, b] or used[b, c] or used[c, a]):
            for x, y in ((a, b), (b, c), (c, a)):
                used[x, y] = used[y, x] = True
            F.append([a, b, c])
    return rng.normal(size=(n_v, 3)), np.array(F)


CASES = [(f"poles of {k} {c}", poles(k, k, c)) for k in (25, 32, 33, 60, 129, 256, 257) for c in (1, 2)]
CASES += [(f"poles of {k}", poles(k, k, 2, 1)) for k in (600, 1025)]
CASES += [("every old vertex of 24 faces", kis(*M.icosphere(2), 2)), ("of 48", kis(*M.icosphere(1), 3)),
          ("fans at one tip", two_fans(40, 1)), ("long fans at one tip", two_fans(150, 2)),
          ("rings that do not fit", edges_of_one_face(60, 3))]


@pytest.mark.parametrize("name,mesh", CASES, ids=[c[0] for c in CASES])
def test_equals_the_oracle(oracle_lib, name, mesh):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F = mesh[0].astype(np.float32), np.ascontiguousarray(mesh[1].astype(np.int32))
    d = torch.device("cuda")
    Vd, Fd = torch.from_numpy(V).to(d), torch.from_numpy(F).to(d)
    print(f"[gpu] qem poles {name} n_f={F.shape[0]}", flush=True)
    g, o = B.qem_edges(Vd, Fd), oracle_lib.qem_edges(V.astype(np.float64), F)
    for x in ("edges", "faces", "valid", "cost", "p"):
        a, b = getattr(g, x).cpu().numpy(), getattr(o, x)
        if x == "p":
            a, b = a[o.valid], b[o.valid]
        np.testing.assert_array_equal(a, b, err_msg=x)
    for target, rounds in ((4, 1), (4, 4), (max(4, F.shape[0] // 3), 1000), (4, 1000)):
        r = B.qem_simplify(Vd, Fd, target, max_rounds=rounds)
        w = oracle_lib.qem_simplify(V, F, target, method="rounds", max_rounds=rounds)
        assert r.rounds == w.rounds, (target, rounds)
        np.testing.assert_array_equal(r.F.cpu().numpy(), w.F)
        np.testing.assert_array_equal(r.V.cpu().numpy(), w.V.astype(np.float32))


def test_rounds_stay_short(capfd):
    """A walk over a pole's faces for each of its neighbours would take n^3 steps of
    one lane a round: minutes for the 1,500 faces here.  A round takes some 4 ms (each
    of a pole's edges tests all of its faces for a turned normal)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F = poles(1500, 7, 2, 12)
    Vd = torch.from_numpy(V.astype(np.float32)).cuda()
    Fd = torch.from_numpy(F.astype(np.int32)).cuda()
    B.qem_simplify(Vd, Fd, len(F) - 100)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    r = B.qem_simplify(Vd, Fd, 500)
    torch.cuda.synchronize()
    ms = 1e3 * (time.perf_counter() - t0)
    with capfd.disabled():
        print(f"[gpu] poles of 1500, {len(F)} faces: {r.rounds} rounds in {ms:.1f} ms", flush=True)
    assert ms < 10 * r.rounds

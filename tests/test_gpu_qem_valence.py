"""Simplification and edge listing where the per-vertex records change form:
vertices of 8, 9, 16, 17 and more faces, rings of more than 16 vertices, fans
with a boundary, soup without shared edges.  Bit for bit the FP64 oracle's,
after one round, after a few and at the end."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from synth import shapes as S  # noqa: E402


def bipyramid(k, layers, seed, boundary=False):
    """Rings of k vertices between two poles of valence k, jittered; without
    the lower pole when `boundary`."""
    rng = np.random.default_rng(seed)
    th = 2 * np.pi * np.arange(k) / k
    V = [[0, 0, 1.3]]
    for r in range(layers):
        z = 0.8 * (1 - 2 * (r + 0.5) / layers)
        w = np.sqrt(1 - z * z)
        V += np.stack([w * np.cos(th + 0.3 * r), w * np.sin(th + 0.3 * r), np.full(k, z)], 1).tolist()
    V += [[0, 0, -1.3]]
    at = lambda r, i: 1 + r * k + i % k  # noqa: E731
    F = [[0, at(0, i), at(0, i + 1)] for i in range(k)]
    for r in range(layers - 1):
        for i in range(k):
            F += [[at(r, i), at(r + 1, i), at(r, i + 1)], [at(r, i + 1), at(r + 1, i), at(r + 1, i + 1)]]
    if not boundary:
        F += [[len(V) - 1, at(layers - 1, i + 1), at(layers - 1, i)] for i in range(k)]
    V = np.array(V) + rng.normal(size=(len(V), 3)) * 0.02
    return V.astype(np.float32), np.array(F, np.int32)


def soup(n, seed):
    rng = np.random.default_rng(seed)
    return rng.normal(size=(3 * n, 3)).astype(np.float32), np.arange(3 * n, dtype=np.int32).reshape(n, 3)


CASES = [(f"bipyramid {k} x {r}{' open' if o else ''}", bipyramid(k, r, k, o)) for k in (8, 9, 16, 17, 24, 40) for r in (1, 5)
         for o in (False, True)] + [("soup", soup(40, 1)), ("patch", tuple(np.asarray(x, t) for x, t in zip(
             S.grid_patch(20, 0.2, 3), (np.float32, np.int32))))]


@pytest.mark.parametrize("name,mesh", CASES, ids=[c[0] for c in CASES])
def test_equals_the_oracle(oracle_lib, name, mesh):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F = mesh
    d = torch.device("cuda")
    Vd, Fd = torch.from_numpy(V).to(d), torch.from_numpy(F).to(d)
    print(f"[gpu] qem valence {name} n_f={F.shape[0]}", flush=True)
    g, o = B.qem_edges(Vd, Fd), oracle_lib.qem_edges(V.astype(np.float64), F)
    for x in ("edges", "faces", "valid", "cost", "p"):
        a, b = getattr(g, x).cpu().numpy(), getattr(o, x)
        if x == "p":
            a, b = a[o.valid], b[o.valid]
        np.testing.assert_array_equal(a, b, err_msg=x)
    for target, rounds in ((4, 1), (4, 3), (max(4, F.shape[0] // 3), 1000), (4, 1000)):
        r = B.qem_simplify(Vd, Fd, target, max_rounds=rounds)
        w = oracle_lib.qem_simplify(V, F, target, method="rounds", max_rounds=rounds)
        assert r.rounds == w.rounds, (target, rounds)
        np.testing.assert_array_equal(r.F.cpu().numpy(), w.F)
        np.testing.assert_array_equal(r.V.cpu().numpy(), w.V.astype(np.float32))

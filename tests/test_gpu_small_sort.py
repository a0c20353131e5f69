"""Codes and sort of small meshes by one workgroup, at the ends of its rounds and of
its range: ascending codes, index order on equal ones, and the same bake bit for
bit as beside a mesh large enough for the passes over many tiles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from synth import meshes as M  # noqa: E402


def _inputs(n, seed, res=64):
    rng = np.random.default_rng(seed)
    V, F = M.icosphere(5)  # 20,480 faces
    V = (V * (1.02 + 0.01 * rng.normal(size=(V.shape[0], 1)))).astype(np.float32)
    F = F[np.sort(rng.permutation(F.shape[0])[:n])]
    if n > 1:
        F[n // 2] = F[0]  # equal codes
    lo_V, lo_F = M.icosphere(1)
    return [torch.as_tensor(np.ascontiguousarray(x)).cuda() for x in
            (V, F.astype(np.int32), M.vertex_normals(V, F), lo_V.astype(np.float32), lo_F.astype(np.int32),
             M.face_grid_atlas(lo_F.shape[0], res))]


@pytest.mark.parametrize("n,bad", [(1, False), (63, False), (1023, True), (1025, False), (4097, False), (8191, True),
                                   (8192, False), (8193, True)])
def test_small_sort(n, bad):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    t = _inputs(n, n)
    if bad:  # a face out of range and a corner that is not a number
        t[1][n // 3, 1] = t[0].shape[0]
        t[0][int(t[1][n // 4, 2])] = float("nan")
    print(f"[gpu] small sort n={n} bad={bad}", flush=True)
    r = B.bake_normals(*t, 64, 0.3)
    torch.cuda.synchronize()
    keys = r.view(B.VIEW_SORTED).view(torch.int32).cpu().numpy().view(np.uint32)[:n].astype(np.int64)
    idx = r.view(B.VIEW_SORTED_IDX).view(torch.int32).cpu().numpy()[:n]
    assert np.array_equal(np.sort(idx), np.arange(n))
    assert np.all(np.diff(keys) >= 0)
    assert np.all(np.diff(idx)[np.diff(keys) == 0] > 0)
    b = B.BakeBatch([(*t, 64, 0.3), (*_inputs(9000, 1), 64, 0.3)])
    b.forward()
    torch.cuda.synchronize()
    assert b.status() == r.status()
    assert (r.status() != 0) == bad
    assert np.array_equal(b.maps[0].cpu().numpy().view(np.uint32), r.map.cpu().numpy().view(np.uint32))
    assert np.array_equal(b.hits[0].cpu().numpy(), r.hit.cpu().numpy())

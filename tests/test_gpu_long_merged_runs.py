"""dL/dhi_N where a vertex has a pair with so many 64-ray batches that its run of
sorted pairs goes on over several groups of 64 and of 256: the runs that a wave
finishes past its own pairs.  Against the FP64 adjoint with the bounds of
test_gpu_backward.py, and bitwise repeatable."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import compare as CMP  # noqa: E402
from synth import Asset  # noqa: E402
from synth import meshes as M  # noqa: E402


# run: pairs that the longest run has at least
@pytest.mark.parametrize("hi_level,res,run", [(0, 256, 65), (0, 512, 257), (0, 1024, 1025), (2, 1024, 129)])
def test_runs_over_groups(oracle_lib, hi_level, res, run):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F = M.icosphere(hi_level)
    hi_V = (V * 1.02).astype(np.float32)
    lo_V, lo_F = M.icosphere(1)
    a = Asset("long runs", hi_V, F.astype(np.int32), M.vertex_normals(hi_V, F), lo_V.astype(np.float32),
              lo_F.astype(np.int32), M.face_grid_atlas(lo_F.shape[0], res), res=res, max_dist=0.4)
    t = B.to_device(a)
    g = torch.from_numpy(np.random.default_rng(res).normal(size=(res, res, 3)).astype(np.float32)).cuda()
    out = []
    for _ in range(2):
        r = B.bake_normals(*t, a.res, a.max_dist, save=True, dilate_passes=0)
        lo, hi = B.bake_normals_backward(r, t, g)
        torch.cuda.synchronize()
        out.append((lo.cpu().numpy(), hi.cpu().numpy()))
    hit = r.hit.cpu().numpy()
    # pairs of a vertex: the batches of 64 rays (in the order of the ray list) that hit one of its faces
    n = int((hit != -3).sum())  # covered texels
    texel = r.view(B.VIEW_RAYS).view(torch.int32).cpu().numpy().reshape(-1, 4)[:n, 0]
    h = hit.reshape(-1)[texel]
    ray = np.nonzero(h >= 0)[0]
    pairs = np.unique((ray // 64)[:, None] * hi_V.shape[0] + F[h[ray]])
    longest = np.bincount(pairs % hi_V.shape[0]).max()
    print(f"[gpu] merged runs hi_v={hi_V.shape[0]} res={res} longest={longest}", flush=True)
    assert longest >= run
    olo, ohi, mlo, mhi, shi = oracle_lib.adjoint_at(a, hit, g.cpu().numpy().astype(np.float64).reshape(-1, 3),
                                                    magnitudes=True, bnoise=CMP.weight_noise(a, hit))
    CMP.compare_grads("lo_V", out[0][0], olo, mlo)
    CMP.compare_grads("hi_N", out[0][1], ohi, mhi, shi)
    assert all(np.array_equal(x.view(np.uint32), y.view(np.uint32)) for x, y in zip(*out))

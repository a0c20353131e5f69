"""dL/dhi_N where many texels hit the same high-poly vertex: its run of sorted
pairs goes on over many waves' groups of 64 (and 256) pairs.  Against the FP64
adjoint with the bounds of test_gpu_backward.py, and bitwise repeatable."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import compare as CMP  # noqa: E402
from synth import Asset  # noqa: E402
from synth import meshes as M  # noqa: E402


# 4,233 rays at 128^2 and 17,733 at 256^2, three pairs each, on 12-162 vertices
@pytest.mark.parametrize("hi_level,res", [(0, 128), (0, 256), (1, 128), (2, 256)])
def test_few_vertices(oracle_lib, hi_level, res):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F = M.icosphere(hi_level)
    hi_V = (V * 1.02).astype(np.float32)
    lo_V, lo_F = M.icosphere(1)
    a = Asset("few vertices", hi_V, F.astype(np.int32), M.vertex_normals(hi_V, F), lo_V.astype(np.float32),
              lo_F.astype(np.int32), M.face_grid_atlas(lo_F.shape[0], res), res=res, max_dist=0.4)
    print(f"[gpu] long runs hi_v={hi_V.shape[0]} res={res}", flush=True)
    t = B.to_device(a)
    g = torch.from_numpy(np.random.default_rng(res).normal(size=(res, res, 3)).astype(np.float32)).cuda()
    out = []
    for _ in range(2):
        r = B.bake_normals(*t, a.res, a.max_dist, save=True, dilate_passes=0)
        lo, hi = B.bake_normals_backward(r, t, g)
        torch.cuda.synchronize()
        out.append((lo.cpu().numpy(), hi.cpu().numpy()))
    hit = r.hit.cpu().numpy()
    assert (hit >= 0).sum() * 3 > 40 * hi_V.shape[0]
    olo, ohi, mlo, mhi, shi = oracle_lib.adjoint_at(a, hit, g.cpu().numpy().astype(np.float64).reshape(-1, 3),
                                                    magnitudes=True, bnoise=CMP.weight_noise(a, hit))
    CMP.compare_grads("lo_V", out[0][0], olo, mlo)
    CMP.compare_grads("hi_N", out[0][1], ohi, mhi, shi)
    assert all(np.array_equal(x.view(np.uint32), y.view(np.uint32)) for x, y in zip(*out))

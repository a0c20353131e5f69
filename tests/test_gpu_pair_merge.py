"""dL/dhi_N through the merged (vertex, sum) pairs of a wave's rays: few and many
vertices a wave, batches without a hit, pairs of many and of no batches in a sort
tile, more batches than one workgroup sums at once, and uneven assets side by
side.  Against the FP64 adjoint with the bounds of test_gpu_backward.py, and
bitwise repeatable."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import compare as CMP  # noqa: E402
from synth import Asset  # noqa: E402
from synth import meshes as M  # noqa: E402


def _asset(hi_level, res, cap, lo_level=1, max_dist=0.4):
    V, F = M.icosphere(hi_level)
    hi_V = (V * 1.02).astype(np.float32)
    N = M.vertex_normals(hi_V, F)
    F = F[V[F][:, :, 2].min(1) > cap]  # the part of the sphere above z = cap
    lo_V, lo_F = M.icosphere(lo_level)
    return Asset("pair merge", hi_V, np.ascontiguousarray(F.astype(np.int32)), N,
                 lo_V.astype(np.float32), lo_F.astype(np.int32), M.face_grid_atlas(lo_F.shape[0], res), res=res,
                 max_dist=max_dist)


def _check(oracle_lib, a, hit, g, lo, hi):
    olo, ohi, mlo, mhi, shi = oracle_lib.adjoint_at(a, hit, g.cpu().numpy().astype(np.float64).reshape(-1, 3),
                                                    magnitudes=True, bnoise=CMP.weight_noise(a, hit))
    CMP.compare_grads("lo_V", lo, olo, mlo)
    CMP.compare_grads("hi_N", hi, ohi, mhi, shi)


# above z = 0.9 most batches have no hit; 512^2 has more than 1,024 batches; level 7
# at 256^2 has more vertices than rays
@pytest.mark.parametrize("hi_level,res,cap", [(5, 512, -2.0), (7, 512, -2.0), (5, 512, 0.9), (7, 256, -2.0),
                                              (0, 512, -2.0), (4, 16, -2.0)])
def test_one_asset(oracle_lib, hi_level, res, cap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    a = _asset(hi_level, res, cap)
    print(f"[gpu] pair merge hi={hi_level} res={res} cap={cap}", flush=True)
    t = B.to_device(a)
    g = torch.from_numpy(np.random.default_rng(res).normal(size=(res, res, 3)).astype(np.float32)).cuda()
    out = []
    for _ in range(2):
        r = B.bake_normals(*t, a.res, a.max_dist, save=True, dilate_passes=0)
        lo, hi = B.bake_normals_backward(r, t, g)
        torch.cuda.synchronize()
        out.append((lo.cpu().numpy(), hi.cpu().numpy()))
    assert r.status() == 0
    _check(oracle_lib, a, r.hit.cpu().numpy(), g, *out[0])
    assert all(np.array_equal(x.view(np.uint32), y.view(np.uint32)) for x, y in zip(*out))


def test_no_hit():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    for res in (128, 512):
        a = _asset(3, res, -2.0, max_dist=1e-4)
        t = B.to_device(a)
        r = B.bake_normals(*t, a.res, a.max_dist, save=True, dilate_passes=0)
        assert not (r.hit >= 0).any()
        lo, hi = B.bake_normals_backward(r, t, torch.ones((res, res, 3), device="cuda"))
        assert not lo.any() and not hi.any()


def test_uneven_assets():
    """Beside others an asset's gradients are those it has by itself."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    assets = [_asset(5, 512, 0.9), _asset(2, 2, -2.0), _asset(3, 128, -2.0, max_dist=1e-4), _asset(6, 256, -2.0),
              _asset(4, 4, -2.0), _asset(0, 512, -2.0)]
    ts = [B.to_device(a) for a in assets]
    gs = [torch.from_numpy(np.random.default_rng(i).normal(size=(a.res, a.res, 3)).astype(np.float32)).cuda()
          for i, a in enumerate(assets)]
    alone = []
    for a, t, g in zip(assets, ts, gs):
        r = B.bake_normals(*t, a.res, a.max_dist, save=True, dilate_passes=0)
        alone.append([x.cpu().numpy() for x in B.bake_normals_backward(r, t, g)])
    batch = B.BakeBatch([tuple(t) + (a.res, a.max_dist) for a, t in zip(assets, ts)], save=True, dilate_passes=0)
    for i, g in enumerate(gs):
        batch.grad_maps[i].copy_(g)
    batch.forward()
    batch.backward()
    torch.cuda.synchronize()
    for i, x in enumerate(alone):
        for u, v in zip(x, (batch.grad_lo_V[i], batch.grad_hi_N[i])):
            assert np.array_equal(u.view(np.uint32), v.cpu().numpy().view(np.uint32)), i

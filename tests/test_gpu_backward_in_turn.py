"""A saved batch of more than 48 x 2^20 texels, whose backward sorts where its
low-poly chain had its terms: both gradients are those of a backward for one alone."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from synth import Asset  # noqa: E402
from synth import meshes as M  # noqa: E402


def test_both_gradients(res=8192):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F = M.icosphere(6)
    lo_V, lo_F = M.icosphere(3)
    a = Asset("in turn", (V * 1.02).astype("f4"), F.astype("i4"), M.vertex_normals(V, F), lo_V.astype("f4"),
              lo_F.astype("i4"), M.face_grid_atlas(lo_F.shape[0], res), res=res, max_dist=0.4)
    t = B.to_device(a)
    print(f"[gpu] backward in turn res={res}", flush=True)
    r = B.bake_normals(*t, res, a.max_dist, save=True, dilate_passes=0)
    assert r.workspace.numel() < 12 << 30
    g = torch.randn((res, res, 3), generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    lo, hi = B.bake_normals_backward(r, t, g)
    lo1, _ = B.bake_normals_backward(r, t, g, need_hi=False)
    _, hi1 = B.bake_normals_backward(r, t, g, need_lo=False)
    torch.cuda.synchronize()
    assert r.status() == 0
    assert (lo != 0).any() and (hi != 0).any()
    assert torch.equal(lo.view(torch.int32), lo1.view(torch.int32))
    assert torch.equal(hi.view(torch.int32), hi1.view(torch.int32))

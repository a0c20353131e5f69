"""The fused fill of uncovered texels against the launches of one pass each, at
images smaller than a tile and with ragged last tiles: a texel filled in pass p
keeps its value in every later one, so k fused passes agree bit for bit with six
separate ones wherever they fill, and fill just the k rings round the coverage.
The bytes are those of the launch that forms them by itself."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from synth import meshes as M  # noqa: E402


def _ring(m):
    p = np.pad(m, 1)
    n = m.shape[0]
    return np.logical_or.reduce([p[i:i + n, j:j + n] for i in range(3) for j in range(3)])


@pytest.mark.parametrize("res,lo_level", [(16, 0), (32, 0), (64, 0), (64, 2), (128, 1), (256, 0), (512, 3)])
def test_fused_passes(res, lo_level):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F = M.icosphere(4)
    hi_V = (V * 1.02).astype(np.float32)
    lo_V, lo_F = M.icosphere(lo_level)
    t = [torch.as_tensor(np.ascontiguousarray(x)).cuda() for x in
         (hi_V, F.astype(np.int32), M.vertex_normals(hi_V, F), lo_V.astype(np.float32), lo_F.astype(np.int32),
          M.face_grid_atlas(lo_F.shape[0], res))]
    print(f"[gpu] fused fill res={res} lo={lo_level}", flush=True)
    ref = B.bake_normals(*t, res, 0.5, dilate_passes=6, rgb8=True)
    want, hit = ref.map.cpu().numpy().view(np.uint32), ref.hit.cpu().numpy().reshape(res, res)
    cov = hit != -3
    assert cov.any() and not cov.all()
    for k in (1, 2, 3, 4):
        cov = _ring(cov)
        r = B.bake_normals(*t, res, 0.5, dilate_passes=k, rgb8=True)
        m = r.map.cpu().numpy().reshape(res, res, 3)
        assert np.array_equal(r.hit.cpu().numpy().reshape(res, res), hit)
        assert np.array_equal(m.view(np.uint32)[cov], want.reshape(res, res, 3)[cov]), k
        assert (m[~cov] == np.array([0, 0, 1], np.float32)).all(), k
        rgb = r.rgb8.cpu().numpy().reshape(res, res, 3)
        assert np.array_equal(rgb[cov], ref.rgb8.cpu().numpy().reshape(res, res, 3)[cov]), k
        assert (rgb[~cov] == np.array([128, 128, 255], np.uint8)).all(), k

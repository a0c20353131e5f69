"""The backprojection maps of many views equal those of the views taken a few
at a time (the kernel keeps 64 view frames at once), and every output value is
written: a texel that no face covers is (-1, -1) and 0."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from synth import meshes as M  # noqa: E402


@pytest.mark.parametrize("res,faces_of_level", [(64, 2), (1, 1), (32, 1)])
def test_views_in_parts(res, faces_of_level):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F, UV = M.textured_bumpy_mesh(level=faces_of_level, res=res)
    eyes = M.sphere_viewpoints(70, [0, 0, 0], 2.5)
    d = torch.device("cuda")
    V, F, UV, E = (torch.from_numpy(x).to(d) for x in (V, F, UV, eyes))
    tan, img = math.tan(math.radians(30.0)), 48

    def maps(a, b, out=None):
        print(f"[gpu] view maps res={res} views {a}-{b}", flush=True)
        return B.view_maps(V, F, UV, res, E[a:b].contiguous(), [0, 0, 0], tan, img, 5.0, 2e-3, out=out)

    # outputs that start as garbage, at an address that is only 4-B aligned
    raw = torch.full((70 * res * res * 3 + 1,), 7.0, device=d)
    n = 70 * res * res
    out = (raw[1:1 + 2 * n].view(70, res, res, 2), raw[1 + 2 * n:].view(70, res, res))
    whole = maps(0, 70, out)
    for a, b in ((0, 1), (10, 20), (60, 70), (64, 70)):
        part = maps(a, b)
        assert torch.equal(part.uv, whole.uv[a:b]) and torch.equal(part.inc, whole.inc[a:b])
    empty = (whole.uv == -1).all(3)
    assert torch.equal(empty.all(0), empty.any(0))  # the eyes see the whole mesh: covered or not is the same in every view
    assert (whole.inc[empty] == 0).all() and (whole.uv != 7.0).all()
    assert int((~empty[0]).sum()) == whole.counter(0)

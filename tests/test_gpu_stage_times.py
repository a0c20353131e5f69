"""Stage times of passes that reuse a slot of the ring of timed passes: a bake whose
low-poly work ran beside the tree build says nothing about the pass after it."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from synth import Asset  # noqa: E402
from synth import meshes as M  # noqa: E402

TAN30 = math.tan(math.radians(30.0))


@pytest.mark.parametrize("which", ["visibility", "view maps"])
def test_after_bakes_beside(which):
    """65 bakes of 81,920 faces fill the ring's 64 slots; then the stages of another
    pass follow one another, so that they add up to the whole."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F = M.icosphere(6)
    lo_V, lo_F = M.icosphere(1)
    a = Asset("stages", V.astype(np.float32), F.astype(np.int32), M.vertex_normals(V, F), lo_V.astype(np.float32),
              lo_F.astype(np.int32), M.face_grid_atlas(lo_F.shape[0], 128), res=128, max_dist=0.4)
    t = B.to_device(a)
    print(f"[gpu] stage times after bakes: {which}", flush=True)
    for _ in range(65):
        B.bake_normals(*t, a.res, a.max_dist, timing=True)
    Vd, Fd = torch.from_numpy(a.hi_V).cuda(), torch.from_numpy(a.hi_F).cuda()
    eyes = torch.from_numpy(M.sphere_viewpoints(8, [0, 0, 0], 2.5).astype(np.float32)).cuda()
    if which == "visibility":
        B.visibility(Vd, Fd, eyes, (0, 0, 0), TAN30, 256, 4.0, timing=True)
    else:
        UV = torch.from_numpy(M.face_grid_atlas(F.shape[0], 1024)).cuda()
        B.view_maps(Vd, Fd, UV, 1024, eyes, (0, 0, 0), TAN30, 256, 5.0, 2e-3, timing=True)
    torch.cuda.synchronize()
    ms = list(B.stage_times().values())
    print("[gpu]", which, [round(x, 4) for x in ms], flush=True)
    # five spans between six events in a row, each reported to some microseconds
    assert abs(sum(ms[:5]) - ms[5]) < 0.03

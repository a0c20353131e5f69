"""The flood fill over hidden fans: many faces around one tip, inside a shell that
sees none or some of them.  Bit for bit the oracle's fill from the same visible faces."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from synth import meshes as M  # noqa: E402

TAN30 = math.tan(math.radians(30.0))


def fan_in_shell(n, holes, flip):
    """A cone of n faces inside an icosphere (with holes), every flip-th inside out."""
    V, F = M.icosphere(4)
    F = F[np.sort(np.random.default_rng(n).permutation(len(F))[holes:])]
    th = 2 * np.pi * np.arange(n) / n
    C = np.concatenate([[[0, 0, 0.3]], np.stack([0.5 * np.cos(th), 0.5 * np.sin(th), 0 * th], 1)])
    fan = np.stack([np.zeros(n, int), 1 + np.arange(n), 1 + (np.arange(n) + 1) % n], 1)
    if flip:
        fan[::flip] = fan[::flip, [0, 2, 1]]
    fan = np.concatenate([fan, [[0, 0, 1], [0, 1, 1]]])  # faces without area share edges too
    return np.concatenate([V, C]).astype(np.float32), np.concatenate([F, len(V) + fan]).astype(np.int32)


def fill(V, F, timing=False):
    import paper_2605_26137_amd.bake as B
    eyes = torch.from_numpy(M.sphere_viewpoints(16, [0, 0, 0], 2.5).astype(np.float32)).cuda()
    r = B.visibility(torch.from_numpy(V).cuda(), torch.from_numpy(F).cuda(), eyes, (0, 0, 0), TAN30, 128, 4.0,
                     timing=timing)
    torch.cuda.synchronize()
    return r


@pytest.mark.parametrize("n,holes,flip", [(64, 0, 0), (300, 100, 0), (300, 100, 7), (3000, 400, 0), (3000, 400, 50)])
def test_equals_the_oracle(oracle_lib, n, holes, flip):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    V, F = fan_in_shell(n, holes, flip)
    print(f"[gpu] flood fans n={n} holes={holes} flip={flip}", flush=True)
    r = fill(V, F)
    vis, ext = r.visible.cpu().numpy(), r.exterior.cpu().numpy()
    assert np.array_equal(ext, np.asarray(oracle_lib.flood_fill(V, F, vis)).astype(bool))


def test_time_follows_the_faces():
    """Each of 20,000 faces walking all of them takes 11 ms; walking the shorter lists,
    half a millisecond."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F = fan_in_shell(20000, 0, 0)
    fill(V, F, timing=True)
    fill(V, F, timing=True)
    ms = list(B.stage_times().values())[3]
    print(f"[gpu] flood fill of a fan of 20,000: {ms:.3f} ms", flush=True)
    assert ms < 5

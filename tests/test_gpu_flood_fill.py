"""The flood fill where it has far to go: a narrow view sees a few faces of a
large patch, and the exterior equals the oracle's fill from those faces."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from synth import meshes as M, shapes as S  # noqa: E402


@pytest.mark.parametrize("faces", ["patch", "shuffled", "flipped half", "folded", "two spheres"])
def test_fill_reaches_far(oracle_lib, faces):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    rng = np.random.default_rng(3)
    if faces == "two spheres":  # one of them far outside the view
        V0, F0 = M.icosphere(4)
        V = np.concatenate([V0, V0 + [9.0, 0, 0]])
        F = np.concatenate([F0, F0 + V0.shape[0]])
    else:
        V, F = S.grid_patch(90, 0.05, 1)  # 16,200 faces
        V = V - 0.5
    if faces == "shuffled":
        F = F[rng.permutation(F.shape[0])]
        p = rng.permutation(V.shape[0])
        V, F = V[np.argsort(p)], p[F]
    if faces == "flipped half":
        F = np.where((V[F].mean(1)[:, :1] > 0.2), F[:, ::-1], F)
    if faces == "folded":
        V = V.copy()
        V[:, 2] += np.where(V[:, 0] > 0.1, 3.0 * (V[:, 0] - 0.1), 0.0)
    V, F = V.astype(np.float32), F.astype(np.int32)
    eye = np.array([[-0.3, -0.2, 2.0]] if faces != "two spheres" else [[0, 0, 2.5]], np.float32)
    target = [-0.3, -0.2, 0.0] if faces != "two spheres" else [0, 0, 0]
    print(f"[gpu] flood fill {faces} n_f={F.shape[0]}", flush=True)
    d = torch.device("cuda")
    out = []
    for _ in range(2):
        r = B.visibility(torch.from_numpy(V).to(d), torch.from_numpy(F).to(d), torch.from_numpy(eye).to(d), target,
                         math.tan(math.radians(0.5)), 32, 5.0)
        assert r.status() == 0
        out.append((r.visible.cpu().numpy(), r.exterior.cpu().numpy()))
    vis, ext = out[0]
    assert 0 < vis.sum() < 60 and ext.sum() > 20 * vis.sum()
    assert np.array_equal(ext, oracle_lib.flood_fill(V, F, vis))
    assert np.array_equal(out[1][0], vis) and np.array_equal(out[1][1], ext)

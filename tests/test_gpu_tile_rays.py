"""Camera rays by pixel blocks: the first hits do not depend on how a launch
cuts its images into blocks (the block side follows from the number of 8 x 8
tiles and the faces per pixel), and agree with the FP64 brute force where the
blocks' lists overflow, on ragged images, from inside the mesh and with a mesh
of a single face."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from compare import check_first_hits  # noqa: E402
from synth import meshes as M  # noqa: E402

TAN30 = math.tan(math.radians(30.0))


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as bake
    bake.lib()
    return bake


def hits(B, V, F, eyes, target, tan_half, res, t_far, count=False):
    print(f"[gpu] tile rays n_f={F.shape[0]} views={eyes.shape[0]} res={res}", flush=True)
    d = torch.device("cuda")
    r = B.visibility(*(torch.from_numpy(np.ascontiguousarray(x, t)).to(d) for x, t in
                       ((V, np.float32), (F, np.int32), (eyes, np.float32))), target, tan_half, res, t_far,
                     first_hit=True, count=count)
    assert r.status() == 0
    return r.first_hit.cpu().numpy(), r


# 33 tiles a side: 256 views take the largest blocks, 8 and 1 smaller ones
@pytest.mark.parametrize("res", [264, 257])
def test_blocks_of_every_side_agree(B, res):
    V, F, _ = M.hidden_face_mesh(outer_level=3, inner_level=2)  # 1,600 faces
    eyes = M.sphere_viewpoints(256, [0, 0, 0], 2.5)
    target = [0.2, -0.1, 0.3]
    every, r = hits(B, V, F, eyes, target, TAN30, res, 4.0)
    assert (every >= 0).mean() > 0.2
    vis = np.zeros(F.shape[0], bool)
    vis[np.unique(every[every >= 0])] = True
    assert np.array_equal(r.visible.cpu().numpy(), vis)
    for lo, n in ((0, 8), (100, 8), (0, 1), (77, 1), (255, 1)):
        some, _ = hits(B, V, F, eyes[lo:lo + n], target, TAN30, res, 4.0)
        assert np.array_equal(some, every[lo:lo + n])
    counted, c = hits(B, V, F, eyes[:8], target, TAN30, res, 4.0, count=True)
    assert np.array_equal(counted, every[:8])
    assert c.counter(1) > 0 and c.counter(2) > 0 and c.counter(3) > 0


@pytest.mark.parametrize("name,level,res,eye,tan_half,t_far", [
    ("lists overflow: 81,920 faces under 24 x 24 pixels", 6, 24, [0.0, 0.1, 2.5], TAN30, 4.0),
    ("one tile and one pixel", 4, 9, [1.9, 1.2, -1.1], TAN30, 4.0),
    ("a single pixel", 4, 1, [0.3, 2.2, 1.0], TAN30, 4.0),
    ("eye inside the mesh", 4, 40, [0.1, -0.3, 0.2], 3.0, 4.0),
    ("range ends inside the mesh", 4, 40, [0.3, 0.2, 2.4], TAN30, 1.45),
    ("a narrow view of a few faces", 3, 64, [0.0, 0.0, 2.5], 1e-3, 4.0),
])
def test_against_brute_force(B, oracle_lib, name, level, res, eye, tan_half, t_far):
    V, F = M.icosphere(level)
    V = M.displace(V, M.noise_radius(M.unit_directions(V), 5, 4, 0.03))
    eyes = np.array([eye, [-1.7, 0.4, 1.6]], np.float32)
    target = [0.05, 0.0, -0.02]
    ids, _ = hits(B, V, F, eyes, target, tan_half, res, t_far)
    P, D = oracle_lib.camera_rays(eyes, target, tan_half, res)
    o_ids, o_t = oracle_lib.first_hit(V, F.astype(np.int32), P, D, t_far, "brute")
    # ragged small images have few rays: any disagreement has to be a tie
    rep = check_first_hits(oracle_lib, V, F.astype(np.int32), P, D, ids, o_ids, o_t, t_far,
                           0.999 if res > 20 else 0.0, "brute")
    print("[gpu]", name, rep, flush=True)
    assert rep.ok(), str(rep)


def test_few_faces(B):
    # no face, a single face (a tree without nodes), a degenerate one beside it
    V = np.array([[-1, -1, 0], [1, -1, 0], [0, 1, 0]], np.float32)
    eyes = np.array([[0, 0, 2], [0, 0, -2]], np.float32)
    for F, face in (([], -1), ([[0, 1, 2]], 0), ([[1, 1, 2], [0, 1, 2]], 1)):
        F = np.array(F, np.int32).reshape(-1, 3)
        ids, _ = hits(B, V, F, eyes, [0, 0, 0], 0.2, 17, 4.0)
        assert (ids[:, 6:10, 6:10] == face).all()
        assert set(np.unique(ids)) <= {-1, face}


def coincident_sheets(n, pitch, seed):
    """Two n x n sheets of quads in z = 0 with the same corners, faces in random
    order, and two far triangles that leave the sheets' faces in one cell of the
    tree's codes (so that the tree splits them by index); partner[f] = the face
    that coincides with f."""
    rng = np.random.default_rng(seed)
    i, j = (x.ravel() for x in np.meshgrid(np.arange(n + 1), np.arange(n + 1), indexing="ij"))
    V = np.stack([(i - n / 2) * pitch, (j - n / 2) * pitch, 0 * i], 1)
    q = (np.arange(n)[:, None] * (n + 1) + np.arange(n)).ravel()
    half = np.concatenate([np.stack([q, q + n + 1, q + 1], 1), np.stack([q + 1, q + n + 1, q + n + 2], 1)])
    order = rng.permutation(2 * len(half))
    place = np.argsort(order)  # where face k of the pair of sheets went
    partner = np.empty(len(order), np.int64)
    partner[place] = np.concatenate([place[len(half):], place[:len(half)]])
    F = np.concatenate([half, half])[order]
    far = 40 * np.array([[-1, -1, -1], [-1, -1.1, -1], [-1.1, -1, -1], [1, 1, 1.1], [1, 1.1, 1], [1.1, 1, 1]]) + 0.02
    F = np.concatenate([F, len(V) + np.arange(6).reshape(2, 3)])
    return (np.concatenate([V, far]).astype(np.float32), F.astype(np.int32),
            np.concatenate([partner, len(partner) + np.arange(2)]))


def test_equal_distances_take_the_lower_index(B, oracle_lib):
    """Coincident faces seen head-on through a narrow lens: some hundred triangles
    in a tile, all at one distance to a few ulp, two at every pixel."""
    t_far = 1.5
    z = 1.0 + np.arange(64) * 1.7e-5
    eyes = np.stack([0 * z, 0 * z, z], 1).astype(np.float32)
    for seed in range(12):
        V, F, partner = coincident_sheets(13, 0.000476, seed)
        ids, r = hits(B, V, F, eyes, [0, 0, 0], 0.001, 8, t_far)
        assert (ids >= 0).all()
        higher = ids > partner[ids]
        print(f"[gpu] coincident sheets {seed}: {higher.sum()} of {ids.size} pixels take the higher index", flush=True)
        assert not higher.any()
        vis = np.zeros(F.shape[0], bool)
        vis[np.unique(ids)] = True
        assert np.array_equal(r.visible.cpu().numpy(), vis)
        P, D = oracle_lib.camera_rays(eyes[:4], [0, 0, 0], 0.001, 8)
        o_ids, o_t = oracle_lib.first_hit(V, F, P, D, t_far, "brute")
        rep = check_first_hits(oracle_lib, V, F, P, D, ids[:4], o_ids, o_t, t_far, 0.9, "brute")
        assert rep.ok(), str(rep)

"""What the framework is measured on: calls a user makes, over the sizes they make them at.

Each case is one pass through the public entry points of `paper_2605_26137_amd.bake`:

  bake        forward bake (ray query), with or without the RGB8 map
  closest     forward bake with the paper's closest-point query
  step        forward with saved state + squared-error loss + backward, through the library's own calls
  train       the same step through torch autograd (BakeNormals)
  batch       several uneven assets, forward + backward in one launch sequence
  visibility  the hidden-face pass
  viewmaps    the backprojection precompute
  simplify    quadric edge-collapse simplification

Inputs are seeded and synthetic: displaced spheres tessellated as cubes of n x n quads a side (12 n^2 faces; other face counts lose
some faces at random, as scans have holes), in a random orientation, low-poly surfaces that follow the high-poly's coarse shape, and
one right-triangle chart a face.  `exact` evaluates the same definitions with plain torch in 64 bits.
"""
import math

import numpy as np
import torch

from paper_2605_26137_amd import bake as B

DEV = "cuda" if torch.cuda.is_available() else "cpu"
TAN_HALF = math.tan(math.radians(30.0))
PAIRS = 1.2e10  # ray-triangle pairs that exact() tries at most


def listed():
    return [
        # the smallest real asset: launch latency decides
        dict(name="bake_128", kind="bake", hi=5120, lo=80, res=128, max_dist=0.1, rgb8=False, dilate=2),
        # a preview-sized bake with the 8-bit map that is written to a texture; ragged counts
        dict(name="bake_512_rgb8", kind="bake", hi=61_403, lo=1_297, res=512, max_dist=0.12, rgb8=True, dilate=4),
        # the paper's own bake: a raw mesh of a million faces onto 5K faces at 1024^2
        dict(name="bake_1024_rgb8", kind="bake", hi=1_000_000, lo=5_000, res=1024, max_dist=0.12, rgb8=True, dilate=2),
        # the paper's correspondence on the headline sizes, rejected beyond 1 % of the box diagonal
        dict(name="closest_2048", kind="closest", hi=1_310_720, lo=20_480, res=2048, max_dist=0.0348, rgb8=False, dilate=2),
        # differentiable bake of a small asset inside a torch training loop
        dict(name="train_256", kind="train", hi=20_000, lo=320, res=256, max_dist=0.1),
        # the headline step
        dict(name="step_2048", kind="step", hi=1_310_720, lo=20_480, res=2048, max_dist=0.12, dilate=2),
        # the largest single bake: the BVH no longer fits the cache
        dict(name="step_4096", kind="step", hi=5_242_880, lo=81_920, res=4096, max_dist=0.15, dilate=2),
        # an uneven batch: 50k-2M faces, three atlas sizes
        dict(name="batch_10", kind="batch", n=10, hi_lo=50_000, hi_hi=2_000_000, lo_lo=1_300, lo_hi=40_000, res_max=2048, spec=0),
        # hidden-face removal at the paper's settings, on a shell with a few holes
        dict(name="visibility_512x1024", kind="visibility", faces=20_165, views=512, res=1024, ids=False),
        # backprojection precompute for the ten texturing views
        dict(name="viewmaps_10x2048", kind="viewmaps", faces=20_480, res=2048, views=10, img=1024, depth=False),
        # the paper's simplification of a raw mesh
        dict(name="simplify_1306800", kind="simplify", faces=1_306_800, target=10_000),
        # the second simplification of an already reduced mesh
        dict(name="simplify_20172", kind="simplify", faces=20_172, target=1_000),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["bake", "bake", "closest", "step", "step", "train", "batch", "visibility", "viewmaps", "simplify"])
    if kind in ("bake", "closest", "step", "train"):
        hi = log(2_000, 300_000 if kind == "train" else 2_000_000)
        lo = min(log(40, 60_000), hi // 4)
        # an atlas has some tens to some thousands of texels a face
        fits = [r for r in (128, 256, 512, 1024, 2048, 4096) if 16 * lo <= r * r <= 16_384 * lo and r <= (1024 if kind == "train" else 4096)]
        c = dict(kind=kind, hi=hi, lo=lo, res=rng.choice(fits or [1024]), max_dist=0.0348 if kind == "closest" else rng.choice([0.1, 0.12, 0.15]))
        if kind != "train":
            c["dilate"] = rng.choice([0, 2, 2, 2, 4, 8])
        if kind in ("bake", "closest"):
            c["rgb8"] = rng.random() < 0.5
        return c
    if kind == "batch":
        return dict(kind=kind, n=rng.randint(2, 16), hi_lo=5_000, hi_hi=log(50_000, 1_000_000), lo_lo=300, lo_hi=log(1_300, 40_000),
                    res_max=rng.choice([512, 1024, 2048]), spec=rng.randrange(1 << 30))
    if kind == "visibility":
        c = dict(kind=kind, faces=log(1_000, 100_000), views=log(8, 512), res=log(96, 800))
        return dict(c, ids=c["views"] * c["res"] ** 2 < 20_000_000 and rng.random() < 0.5)
    if kind == "viewmaps":
        return dict(kind=kind, faces=log(1_000, 60_000), res=rng.choice([512, 1024, 2048]), views=rng.randint(4, 12), img=log(256, 1536), depth=rng.random() < 0.5)
    n = log(20, 330)
    return dict(kind="simplify", faces=12 * n * n, target=max(200, int(12 * n * n / math.exp(rng.uniform(math.log(2), math.log(130))))))


# ---- inputs ------------------------------------------------------------------------------------------------------------------


def _gen(*key):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(np.random.SeedSequence([int(k) for k in key]).generate_state(1, np.uint64)[0] >> 1))
    return g


def _rotation(g):
    q, _ = torch.linalg.qr(torch.randn(3, 3, generator=g, device=DEV, dtype=torch.float64).cpu())
    return (q * torch.det(q)).to(DEV)  # never a mirror image


def _sphere(faces, g):
    """Unit directions [n_v, 3] f64 and faces [faces, 3] i64 of a cube of n x n quads a side, spread evenly by angle."""
    n = max(1, math.isqrt(max(0, faces - 1) // 12) + 1)
    i, j = torch.meshgrid(torch.arange(n, device=DEV), torch.arange(n, device=DEV), indexing="ij")
    i, j = i.reshape(-1), j.reshape(-1)
    quads = []
    for axis in range(3):
        for side in (0, n):
            def key(a, b):
                c = [None] * 3
                c[axis], c[(axis + 1) % 3], c[(axis + 2) % 3] = torch.full_like(a, side), a, b
                return (c[0] * (n + 1) + c[1]) * (n + 1) + c[2]
            k = [key(i, j), key(i + 1, j), key(i + 1, j + 1), key(i, j + 1)]
            quads.append(torch.stack(k if side else k[::-1], 1))
    quads = torch.cat(quads)
    keys, q = torch.unique(quads, return_inverse=True)
    F = torch.stack([q[:, [0, 1, 2]], q[:, [0, 2, 3]]], 1).reshape(-1, 3)
    p = torch.stack([keys // (n + 1) ** 2, keys // (n + 1) % (n + 1), keys % (n + 1)], 1).double()
    p = torch.tan((p * (2.0 / n) - 1.0) * (math.pi / 4))
    U = p / p.norm(dim=1, keepdim=True)
    if F.shape[0] > faces:
        F = F[torch.randperm(F.shape[0], generator=g, device=DEV)[:faces].sort().values]
    return (U[:, :1] * (R := _rotation(g))[0] + U[:, 1:2] * R[1] + U[:, 2:] * R[2]), F


class _Surface:
    """r(u) = 1 + four octaves of seeded waves (+ bumps)."""

    def __init__(self, g, bumps=0):
        d = torch.randn(4, 8, 3, generator=g, device=DEV, dtype=torch.float64)
        self.k = d / d.norm(dim=2, keepdim=True) * (3 * math.pi * 2.0 ** torch.arange(4, device=DEV, dtype=torch.float64))[:, None, None]
        self.p = 2 * math.pi * torch.rand(4, 8, generator=g, device=DEV, dtype=torch.float64)
        c = torch.randn(bumps, 3, generator=g, device=DEV, dtype=torch.float64)
        self.c = c / c.norm(dim=1, keepdim=True)

    def at(self, U, octaves=4):
        r = torch.ones(U.shape[0], device=DEV, dtype=torch.float64)
        for o in range(octaves):
            for w in range(8):
                k = self.k[o, w]
                r += 0.006 * 0.5 ** o * torch.cos(U[:, 0] * k[0] + U[:, 1] * k[1] + U[:, 2] * k[2] + self.p[o, w])
        for c in self.c:
            r += 0.08 * torch.exp(((U - c) ** 2).sum(1) / (-2 * 0.06 ** 2))
        return r


def _normals(V, F):
    """Area-weighted unit vertex normals, summed in whole numbers: the same in any order."""
    a, b, c = (V[F[:, k]].double() for k in range(3))
    n = (torch.cross(b - a, c - a, dim=1) * (F.shape[0] * 2.0 ** 32)).round().long()
    s = torch.zeros(V.shape[0], 3, dtype=torch.int64, device=DEV)
    for k in range(3):
        s.index_add_(0, F[:, k], n)
    s = s.double()
    return (s / s.norm(dim=1, keepdim=True).clamp_min(1e-300)).float()


def _atlas(faces, res):
    """Per-corner UVs: face f in cell (f mod G, f div G) of a G x G grid, padded by two texels or a quarter of the cell."""
    G = math.isqrt(max(0, faces - 1)) + 1
    s = res / G
    p = min(2.0, s / 4)
    f = torch.arange(faces, device=DEV)
    x0, y0 = (f % G).double() * s, (f // G).double() * s
    x = torch.stack([x0 + p, x0 + s - p, x0 + p], 1)
    y = torch.stack([y0 + p, y0 + p, y0 + s - p], 1)
    return (torch.stack([x, y], 2) / res).float().contiguous()


def _asset(hi, lo, res, seed, k=0):
    """(hi_V, hi_F, hi_N, lo_V, lo_F, lo_UV)."""
    g = _gen(seed, k, 1)
    S = _Surface(g)
    U, F = _sphere(hi, g)
    hi_V, hi_F = (U * S.at(U)[:, None]).float(), F
    U, F = _sphere(lo, g)
    lo_V = (U * S.at(U, 2)[:, None]).float()
    return hi_V, hi_F.int(), _normals(hi_V, hi_F), lo_V, F.int().contiguous(), _atlas(F.shape[0], res)


def _eyes(views, seed):
    """Camera positions spread over the sphere of radius 2.5, turned at random."""
    k = np.arange(views)
    z = 1 - (2 * k + 1) / views
    phi = k * math.pi * (3 - math.sqrt(5.0))
    P = torch.from_numpy(np.stack([np.sqrt(1 - z * z) * np.cos(phi), np.sqrt(1 - z * z) * np.sin(phi), z], 1) * 2.5)
    return (P @ _rotation(_gen(seed, 2)).cpu()).float().to(DEV)


def _batch_specs(c):
    rng = np.random.default_rng(c["spec"])

    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    return [(log(c["hi_lo"], c["hi_hi"]), log(c["lo_lo"], c["lo_hi"]), int(c["res_max"] >> rng.integers(0, 3))) for _ in range(c["n"])]


def _empty(n):
    return torch.empty(n, dtype=torch.uint8, device=DEV)


def _inputs(c, seed):
    """The tensors of a case: what prepare() and exact() both start from."""
    s = dict(c)
    if c["kind"] in ("bake", "closest", "step", "train"):
        s["mesh"] = _asset(c["hi"], c["lo"], c["res"], seed)
        if c["kind"] in ("step", "train"):
            t = torch.randn(c["res"], c["res"], 3, generator=_gen(seed, 3), device=DEV) * 0.3
            t[..., 2] += 1
            s["target"] = t / (t * t).sum(2, keepdim=True).sqrt()
    elif c["kind"] == "batch":
        s["meshes"] = [(*_asset(h, l, r, seed, k), r, 0.1) for k, (h, l, r) in enumerate(_batch_specs(c))]
        s["grads"] = [torch.randn(m[6], m[6], 3, generator=_gen(seed, k, 4), device=DEV) for k, m in enumerate(s["meshes"])]
    elif c["kind"] == "visibility":
        g = _gen(seed, 1)
        U, F = _sphere(c["faces"], g)
        Ui, Fi = _sphere(max(12, c["faces"] // 16), g)  # a sphere inside that no camera sees
        s["V"] = torch.cat([U * _Surface(g).at(U)[:, None], Ui * 0.55]).float()
        s["F"] = torch.cat([F, Fi + U.shape[0]]).int()
        s["eyes"] = _eyes(c["views"], seed)
    elif c["kind"] == "viewmaps":
        g = _gen(seed, 1)
        U, F = _sphere(c["faces"], g)
        s["V"], s["F"] = (U * _Surface(g, 32).at(U)[:, None]).float(), F.int().contiguous()
        s["UV"], s["eyes"] = _atlas(F.shape[0], c["res"]), _eyes(c["views"], seed)
    else:
        g = _gen(seed, 1)
        U, F = _sphere(c["faces"], g)
        s["V"], s["F"] = (U * _Surface(g).at(U)[:, None]).float(), F.int().contiguous()
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    k = case["kind"]
    if k in ("bake", "closest", "step"):
        hi_V, hi_F, _, lo_V, lo_F, _ = s["mesh"]
        o = B.make_options(case["dilate"], k == "step", query="closest" if k == "closest" else "ray")
        s["ws"] = _empty(B.workspace_size(hi_V.shape[0], hi_F.shape[0], lo_V.shape[0], lo_F.shape[0], case["res"], o))
    elif k == "train":
        m = list(s["mesh"])
        m[2].requires_grad_(True)
        m[3].requires_grad_(True)
    elif k == "batch":
        s["batch"] = B.BakeBatch(s["meshes"], save=True)
        for dst, src in zip(s["batch"].grad_maps, s.pop("grads")):
            dst.copy_(src)
    elif k == "visibility":
        s["ws"] = _empty(B.visibility_workspace_size(s["V"].shape[0], s["F"].shape[0]))
    elif k == "viewmaps":
        s["ws"] = _empty(B.view_maps_workspace_size(s["V"].shape[0], s["F"].shape[0], case["res"], case["views"], case["img"]))
    else:
        s["ws"] = _empty(B.qem_workspace_size(s["V"].shape[0], s["F"].shape[0]))
    return s


def run(s):
    k = s["kind"]
    if k in ("bake", "closest"):
        r = B.bake_normals(*s["mesh"], s["res"], s["max_dist"], dilate_passes=s["dilate"], rgb8=s["rgb8"], query="ray" if k == "bake" else k, workspace=s["ws"])
        return [r.map, r.hit, r.rgb8] if s["rgb8"] else [r.map, r.hit]
    if k == "step":
        r = B.bake_normals(*s["mesh"], s["res"], s["max_dist"], dilate_passes=s["dilate"], save=True, workspace=s["ws"])
        loss, grad = B.sq_loss(r.map, s["target"])
        lo, hi = B.bake_normals_backward(r, s["mesh"], grad)
        return [r.map, r.hit, loss, lo, hi]
    if k == "train":
        hi_V, hi_F, hi_N, lo_V, lo_F, lo_UV = s["mesh"]
        m, hit = B.BakeNormals.apply(lo_V, hi_N, hi_V, hi_F, lo_F, lo_UV, s["res"], s["max_dist"])
        lo, hi = torch.autograd.grad(((m - s["target"]) ** 2).sum(), (lo_V, hi_N))
        return [m.detach(), hit, lo, hi]
    if k == "batch":
        b = s["batch"]
        b.forward()
        b.backward()
        return [x for t in zip(b.maps, b.hits, b.grad_lo_V, b.grad_hi_N) for x in t]
    if k == "visibility":
        r = B.visibility(s["V"], s["F"], s["eyes"], (0, 0, 0), TAN_HALF, s["res"], 4.0, first_hit=s["ids"], workspace=s["ws"])
        return [r.visible, r.exterior, r.first_hit] if s["ids"] else [r.visible, r.exterior]
    if k == "viewmaps":
        r = B.view_maps(s["V"], s["F"], s["UV"], s["res"], s["eyes"], (0, 0, 0), TAN_HALF, s["img"], 5.0, 2e-3, depth=s["depth"], workspace=s["ws"])
        return [r.uv, r.inc, r.depth] if s["depth"] else [r.uv, r.inc]
    r = B.qem_simplify(s["V"], s["F"], s["target"], workspace=s["ws"])
    return [r.V, r.F, r.rounds]


def work(case):
    """Bytes: every input read and every output written once.  Flops: setting up each ray or texel and one test of the triangle it
    finds (about 150), as much again for its gradient, and about 500 for each edge that a simplification takes away."""
    k = case["kind"]

    def one(hi, lo, res, grad, extra=0):
        tex = res * res
        rays = tex // 2
        b = 12 * (hi + 2 * hi // 2) + 12 * lo + 6 * lo + 24 * lo + 16 * tex + extra
        if grad:
            b += 24 * tex + 6 * hi + 6 * lo
        return b, rays * 150 * (2 if grad else 1)

    if k in ("bake", "closest"):
        b, f = one(case["hi"], case["lo"], case["res"], False, 3 * case["res"] ** 2 if case["rgb8"] else 0)
    elif k in ("step", "train"):
        b, f = one(case["hi"], case["lo"], case["res"], True)
    elif k == "batch":
        b, f = map(sum, zip(*(one(h, l, r, True) for h, l, r in _batch_specs(case))))
    elif k == "visibility":
        rays = case["views"] * case["res"] ** 2
        b, f = 20 * case["faces"] + (4 * rays if case["ids"] else 0), 150 * rays
    elif k == "viewmaps":
        rays = case["views"] * case["img"] ** 2
        b = 42 * case["faces"] + 12 * case["views"] * case["res"] ** 2 + (4 * rays if case["depth"] else 0)
        f = 150 * rays + 30 * case["views"] * case["res"] ** 2
    else:
        b, f = 18 * (case["faces"] + case["target"]), 750 * (case["faces"] - case["target"])
    return {"bytes": int(b), "flops": int(f)}


# ---- the same results in 64 bits ----------------------------------------------------------------------------------------------

EDGE_EPS, BINS = 2.0 ** -14, 2.0 ** 20


def _dot(a, b):
    return (a * b).sum(-1)


def _unit(a):
    return a / a.norm(dim=-1, keepdim=True)


def _raster(UV, res):
    """Covered texels and their faces and exact barycentric weights; the lowest face has a texel that several cover."""
    q = (UV.double() * (res * 256.0)).round().long()
    X, Y = q[..., 0], q[..., 1]
    j0, i0 = (X.amin(1) + 127) // 256, (Y.amin(1) + 127) // 256
    w = int(max(((X.amax(1) - 128) // 256 - j0).max(), ((Y.amax(1) - 128) // 256 - i0).max())) + 1
    faces = torch.full((res * res,), 1 << 40, dtype=torch.int64, device=DEV)
    found = []
    for f0 in range(0, UV.shape[0], max(1, 20_000_000 // (w * w))):
        f = torch.arange(f0, min(UV.shape[0], f0 + max(1, 20_000_000 // (w * w))), device=DEV)
        d = torch.arange(w, device=DEV)
        i = (i0[f][:, None, None] + d[None, :, None]).expand(-1, w, w)
        j = (j0[f][:, None, None] + d[None, None, :]).expand(-1, w, w)
        cx, cy = 256 * j + 128, 256 * i + 128
        x, y = ([t[f, k][:, None, None] for k in range(3)] for t in (X, Y))
        E = [(x[b] - x[a]) * (cy - y[a]) - (y[b] - y[a]) * (cx - x[a]) for a, b in ((1, 2), (2, 0), (0, 1))]
        S = E[0] + E[1] + E[2]
        ok = ((E[0] >= 0) & (E[1] >= 0) & (E[2] >= 0) | (E[0] <= 0) & (E[1] <= 0) & (E[2] <= 0)) & (S != 0) & (i >= 0) & (j >= 0) & (i < res) & (j < res)
        fb = f[:, None, None].expand(-1, w, w)[ok]
        t = (i * res + j)[ok]
        faces.scatter_reduce_(0, t, fb, "amin")
        found.append((t, fb, torch.stack([e[ok] for e in E], 1).double() / S[ok].double()[:, None]))
    t, f, b = (torch.cat(x) for x in zip(*found))
    keep = faces[t] == f
    return t[keep], f[keep], b[keep]


def _frames(V, F, UV, res):
    """Unit vertex normals, face tangents and handedness, differentiable in V."""
    q = (UV.double() * (res * 256.0)).round()
    du, dv = (q[:, 1:] - q[:, :1]).unbind(2)
    a, b, c = (V[F[:, k]] for k in range(3))
    e1, e2 = b - a, c - a
    n = torch.cross(e1, e2, dim=1)
    sn = torch.zeros_like(V)
    for k in range(3):
        sn = sn.index_add(0, F[:, k], n)
    sg = torch.sign(du[:, 0] * dv[:, 1] - du[:, 1] * dv[:, 0])[:, None]
    T = sg * (e1 * dv[:, 1:] - e2 * dv[:, :1])
    Bt = sg * (e2 * du[:, :1] - e1 * du[:, 1:])
    h = torch.where(_dot(torch.cross(n, T, dim=1), Bt) < 0, -1.0, 1.0).double().detach()
    return sn / sn.norm(dim=1, keepdim=True).clamp_min(1e-300), T, h


def _first(P, D, V, F, far, line):
    """The face of the least (distance bin, index) on each line within +-far (or half-line within far), or -1; and its distance."""
    a, b, c = (V[F[:, k]] for k in range(3))
    n = torch.cross(b - a, c - a, dim=1)
    edges = [torch.cat([torch.cross(p, q, dim=1), q - p], 1).T.contiguous() for p, q in ((b, c), (c, a), (a, b))]
    nT, na = n.T.contiguous(), _dot(n, a)
    best = torch.full((P.shape[0],), 1 << 62, dtype=torch.int64, device=DEV)
    step = max(1, 100_000_000 // max(1, F.shape[0]))
    idx = torch.arange(F.shape[0], device=DEV)
    for r in range(0, P.shape[0], step):
        p, d = P[r:r + step], D[r:r + step]
        L = torch.cat([d, torch.cross(p, d, dim=1)], 1)
        s = [L @ e for e in edges]
        S = s[0] + s[1] + s[2]
        low = torch.minimum(torch.minimum(s[0] / S, s[1] / S), s[2] / S)
        t = (na - p @ nT) / (d @ nT)
        ok = (low >= -EDGE_EPS) & ((t.abs() <= far) if line else (t > 0) & (t <= far))
        key = torch.where(ok, (t.abs() * (BINS / far)).floor(), 0.0).long() * (1 << 31) + idx
        best[r:r + step] = torch.where(ok, key, 1 << 62).amin(1)
    hit = torch.where(best < 1 << 62, best % (1 << 31), -1)
    g = hit.clamp_min(0)
    return hit, (na[g] - _dot(P, n[g])) / _dot(D, n[g])


def _segment(p, a, b):
    return (_dot(p - a, b - a) / _dot(b - a, b - a)).clamp(0, 1)


def _closest(P, V, F, far):
    """The face of the least (distance bin, index) around each point within far, or -1, and its nearest point's weights."""
    a, b, c = (V[F[:, k]] for k in range(3))
    n = _unit(torch.cross(b - a, c - a, dim=1))
    cor = [(a, b), (b, c), (c, a)]
    best = torch.full((P.shape[0],), 1 << 62, dtype=torch.int64, device=DEV)
    step = max(1, 50_000_000 // max(1, F.shape[0]))
    idx = torch.arange(F.shape[0], device=DEV)
    for r in range(0, P.shape[0], step):
        p = P[r:r + step]
        h = p @ n.T - _dot(n, a)
        inside, near = torch.ones_like(h, dtype=torch.bool), None
        for u, v in cor:
            m = torch.cross(n, v - u, dim=1)
            inside &= p @ m.T - _dot(m, u) >= 0
            e = v - u
            t = ((p @ e.T - _dot(u, e)) / _dot(e, e)).clamp(0, 1)
            pu = _dot(p, p)[:, None] - 2 * (p @ u.T) + _dot(u, u)
            d2 = pu - 2 * t * (p @ e.T - _dot(u, e)) + t * t * _dot(e, e)
            near = d2 if near is None else torch.minimum(near, d2)
        d = torch.where(inside, h.abs(), near.clamp_min(0).sqrt())
        key = (d * (BINS / far)).floor().clamp_max(2.0 ** 30).long() * (1 << 31) + idx
        best[r:r + step] = torch.where(d <= far, key, 1 << 62).amin(1)
    hit = torch.where(best < 1 << 62, best % (1 << 31), -1)
    g = hit.clamp_min(0)
    a, b, c, n = a[g], b[g], c[g], n[g]
    area = _dot(torch.cross(b - a, c - a, dim=1), n)
    w = torch.stack([_dot(torch.cross(y - x, P - x, dim=1), n) for x, y in ((b, c), (c, a), (a, b))], 1) / area[:, None]
    ts = torch.stack([_segment(P, x, y) for x, y in ((a, b), (b, c), (c, a))], 1)
    ds = torch.stack([(x + ts[:, k:k + 1] * (y - x) - P).norm(dim=1) for k, (x, y) in enumerate(((a, b), (b, c), (c, a)))], 1)
    k = ds.argmin(1)
    t = ts.gather(1, k[:, None])
    one = torch.eye(3, dtype=torch.float64, device=DEV)
    return hit, torch.where((w >= 0).all(1, keepdim=True), w, one[k] * (1 - t) + one[(k + 1) % 3] * t)


def _dilate(m, filled, passes):
    """Each pass fills every empty texel beside filled ones with the normalised sum of those."""
    res = m.shape[0]
    for _ in range(passes):
        v = torch.zeros(res + 2, res + 2, 3, dtype=torch.float64, device=DEV)
        v[1:-1, 1:-1] = torch.where(filled[..., None], m, 0.0)
        s = sum(v[1 + y:res + 1 + y, 1 + x:res + 1 + x] for y in (-1, 0, 1) for x in (-1, 0, 1) if x or y)
        l = s.norm(dim=2, keepdim=True)
        new = ~filled & (l[..., 0] > 0)
        m = torch.where(new[..., None], s / l.clamp_min(1e-300), m)
        filled = filled | new
    return m


def _bake64(mesh, res, far, closest=False, grad=False):
    """The baked map before dilation, its covered texels, and lo_V and hi_N as it was made from them."""
    hi_V, hi_F, hi_N, lo_V, lo_F, UV = (x.detach() for x in mesh)
    V, F, N, lV, lF = hi_V.double(), hi_F.long(), hi_N.double(), lo_V.double(), lo_F.long()
    lV.requires_grad_(grad)
    N.requires_grad_(grad)
    t, f, w = _raster(UV, res)
    n, T, h = _frames(lV, lF, UV, res)
    P, M = (sum(w[:, k:k + 1] * x[lF[f, k]] for k in range(3)) for x in (lV, n))
    D = M / M.norm(dim=1, keepdim=True)
    if closest:
        hit, beta = _closest(P.detach(), V, F, far)
        c = F[hit.clamp_min(0)]
    else:
        hit, _ = _first(P.detach(), D.detach(), V, F, far, True)
        c = F[hit.clamp_min(0)]
        v = [V[c[:, k]] - P for k in range(3)]
        s = torch.stack([_dot(D, torch.cross(v[a], v[b], dim=1)) for a, b in ((1, 2), (2, 0), (0, 1))], 1)
        beta = s / s.sum(1, keepdim=True)
    H = sum(beta[:, k:k + 1] * N[c[:, k]] for k in range(3))
    H = H / H.norm(dim=1, keepdim=True)
    Tp = _unit(T[f] - D * _dot(T[f], D)[:, None])
    Bp = torch.cross(D, Tp, dim=1) * h[f][:, None]
    out = torch.stack([_dot(H, Tp), _dot(H, Bp), _dot(H, D)], 1)
    up = torch.tensor([0.0, 0.0, 1.0], dtype=torch.float64, device=DEV)
    m = up.expand(res * res, 3).index_put((t,), torch.where((hit >= 0)[:, None], out, up)).reshape(res, res, 3)
    filled = torch.zeros(res * res, dtype=torch.bool, device=DEV)
    filled[t] = True
    return m, filled.reshape(res, res), lV, N


def _frame_of(eye):
    f = _unit(-eye)
    a = torch.zeros(3, dtype=torch.float64, device=DEV)
    a[int(eye.abs().argmin())] = 1
    r = _unit(torch.cross(f, a, dim=0))
    return f, r, torch.cross(r, f, dim=0)


def _maps64(s):
    V, F, res, img = s["V"].double(), s["F"].long(), s["res"], s["img"]
    t, f, w = _raster(s["UV"], res)
    n = _frames(V, F, s["UV"], res)[0]
    P = sum(w[:, k:k + 1] * V[F[f, k]] for k in range(3))
    N = _unit(sum(w[:, k:k + 1] * n[F[f, k]] for k in range(3)))
    rays = s["views"] * img * img * F.shape[0] <= PAIRS
    UVs = torch.full((s["views"], res * res, 2), -1.0, dtype=torch.float64, device=DEV)
    inc = torch.zeros(s["views"], res * res, dtype=torch.float64, device=DEV) if rays else None
    depth = torch.zeros(s["views"], img, img, dtype=torch.float64, device=DEV) if rays else None
    for k, e in enumerate(s["eyes"].double()):
        fw, r, u = _frame_of(e)
        q = P - e
        z = q @ fw
        col = (q @ r / (z * TAN_HALF) + 1) * img / 2 - 0.5
        row = (1 - q @ u / (z * TAN_HALF)) * img / 2 - 0.5
        ok = (z > 0) & (col >= -0.5) & (col < img - 0.5) & (row >= -0.5) & (row < img - 0.5)
        UVs[k, t[ok]] = torch.stack([col, row], 1)[ok]
        if rays:
            c = ((torch.arange(img, device=DEV) + 0.5).double() * 2 / img - 1) * TAN_HALF
            D = _unit(fw + (c[None, :, None] * r - c[:, None, None] * u).reshape(-1, 3))
            hit, far = _first(e.expand_as(D), D, V, F, 5.0, False)
            zb = torch.where(hit >= 0, far * (D @ fw), math.inf)
            depth[k] = torch.where(hit >= 0, far, 0.0).reshape(img, img)
            px = ((row + 0.5).floor().long() * img + (col + 0.5).floor().long())[ok]
            seen = z[ok] <= zb[px] + 2e-3
            inc[k, t[ok]] = torch.where(seen, _dot(N, _unit(-q))[ok].clamp_min(0), 0.0)
    out = [UVs.reshape(-1, res, res, 2), inc.reshape(-1, res, res) if rays else None]
    return out + [None] if s["depth"] else out


def exact(case, seed):
    k = case["kind"]
    if k in ("visibility", "simplify"):  # whole numbers; positions after thousands of dependent decisions
        return None
    if k == "viewmaps":
        return _maps64(_inputs(case, seed))
    if k == "batch":
        if sum(r * r / 2 * h for h, _, r in _batch_specs(case)) > PAIRS:
            return None
        s, out = _inputs(case, seed), []
        for m, g in zip(s["meshes"], s["grads"]):
            a, filled, lV, N = _bake64(m[:6], m[6], m[7], grad=True)
            lo, hi = torch.autograd.grad(a, (lV, N), g.double())
            out += [_dilate(a.detach(), filled, 2), None, lo, hi]
        return out
    if case["res"] ** 2 / 2 * case["hi"] > (PAIRS / 8 if k == "closest" else PAIRS):
        return None
    s = _inputs(case, seed)
    m, filled, lV, N = _bake64(s["mesh"], case["res"], case["max_dist"], k == "closest", k in ("step", "train"))
    if k in ("bake", "closest"):
        m = _dilate(m, filled, case["dilate"])
        return [m, None, None] if case["rgb8"] else [m, None]
    if k == "step":  # the loss is of the dilated map, its gradient is taken at every texel and reaches the covered ones
        d = _dilate(m.detach(), filled, case["dilate"])
        diff = d - s["target"].double()
        lo, hi = torch.autograd.grad(m, (lV, N), 2 * diff)
        return [d, None, (diff * diff).sum().reshape(1), lo, hi]
    lo, hi = torch.autograd.grad(((m - s["target"].double()) ** 2).sum(), (lV, N))
    return [m.detach(), None, lo, hi]

"""The hierarchy at the sizes where its tiles (1,024 leaves) and the joins of
their lists (64 lists, 128 for the last join) begin and end, against the radix
tree formed on the host from the sorted codes: the same children at the same
node indices, and boxes that hold the leaves' triangles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from synth import meshes as M  # noqa: E402
from test_gpu_parity import decode_nodes  # noqa: E402


def radix_tree(keys):
    """Children of every node [n-1, 2] (~leaf for leaves), and the nodes with
    parents before children."""
    n = len(keys)
    k = (keys.astype(np.uint64) << np.uint64(32)) | np.arange(n, dtype=np.uint64)
    x = k[1:] ^ k[:-1]  # the largest difference of a range marks its split
    refs = np.zeros((n - 1, 2), np.int64)
    order, todo = [], [(0, n - 1, 0)]
    best = _range_argmax(x)
    while todo:
        lo, hi, at = todo.pop()
        s = best(lo, hi)
        refs[at] = ~s if s == lo else s, ~(s + 1) if s + 1 == hi else s + 1
        order.append(at)
        if s > lo:
            todo.append((lo, s, s))
        if s + 1 < hi:
            todo.append((s + 1, hi, s + 1))
    return refs, order


def _range_argmax(x):
    rows = [np.arange(len(x))]
    while 2 << (len(rows) - 1) <= len(x):
        h, p = 1 << (len(rows) - 1), rows[-1]
        a, b = p[:-h], p[h:]
        rows.append(np.where(x[a] >= x[b], a, b))

    def best(lo, hi):
        j = (hi - lo).bit_length() - 1
        a, b = rows[j][lo], rows[j][hi - (1 << j)]
        return int(a if x[a] >= x[b] else b)
    return best


@pytest.mark.parametrize("n,kind", [(1, "soup"), (2, "soup"), (3, "equal"), (1023, "soup"), (1024, "soup"),
                                    (1025, "soup"), (2049, "equal"), (65536, "soup"), (65537, "equal"),
                                    (131072, "chain"), (131073, "soup")])
def test_radix_tree(n, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    rng = np.random.default_rng(n)
    if kind == "equal":      # one code: the order of the faces decides
        c = np.zeros((n, 3))
    elif kind == "chain":    # halving distances: the deepest codes
        c = np.ldexp(1.0, -rng.integers(0, 12, n))[:, None] * rng.choice([1.0, -1.0], (n, 3))
    else:
        c = rng.uniform(-1, 1, (n, 3))
    d = 0.01 * rng.normal(size=(n, 3, 3))
    V = (c[:, None] + (d - d.mean(1, keepdims=True) if kind != "equal" else 0 * d)).reshape(-1, 3).astype(np.float32)
    F = np.arange(3 * n, dtype=np.int32).reshape(n, 3)
    N = np.tile(np.array([0, 0, 1], np.float32), (3 * n, 1))
    lo_V, lo_F = M.icosphere(0)
    uv = M.face_grid_atlas(lo_F.shape[0], 32)
    ws = torch.full((B.workspace_size(3 * n, n, lo_V.shape[0], lo_F.shape[0], 32),), 255, dtype=torch.uint8,
                    device="cuda")
    t = [torch.as_tensor(np.ascontiguousarray(x)).cuda() for x in
         (V, F, N, lo_V.astype(np.float32), lo_F.astype(np.int32), uv)]
    print(f"[gpu] tree n={n} {kind}", flush=True)
    r = B.bake_normals(*t, 32, 0.1, workspace=ws)
    torch.cuda.synchronize()
    assert r.status() == 0
    ids = r.view(B.VIEW_LEAVES).view(torch.float32).cpu().numpy().reshape(-1, 12)[:n, 9].copy().view(np.int32)
    assert np.array_equal(np.sort(ids), np.arange(n))
    if n == 1:
        return
    keys = r.view(B.VIEW_SORTED).view(torch.int32).cpu().numpy().view(np.uint32)[:n]
    raw = r.view(B.VIEW_NODES).view(torch.int32).cpu().numpy().reshape(-1, 8)[:n - 1]
    lo, hi, refs, _ = decode_nodes(raw)
    want, order = radix_tree(keys)
    assert np.array_equal(refs, want)
    tri = V[F[ids]]
    leaf = np.stack([tri.min(1), tri.max(1)], 1)
    box = np.zeros((n - 1, 2, 3), np.float32)
    for p in reversed(order):
        b = [leaf[~c] if c < 0 else box[c] for c in want[p]]
        box[p] = np.minimum(b[0][0], b[1][0]), np.maximum(b[0][1], b[1][1])
        for j in range(2):
            assert (lo[p, j] <= b[j][0]).all() and (hi[p, j] >= b[j][1]).all(), (p, j)

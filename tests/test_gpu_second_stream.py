"""Bakes and view maps of few faces with and without the second stream: a call takes
it when the one before it came from the same stream, so the first call, its
repeats, calls from alternating streams and a captured batch give the same bits,
with the workspace poisoned in between."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from synth import meshes as M  # noqa: E402


def _mesh(n):
    V, F = M.icosphere(5)
    V = (V * 1.02).astype(np.float32)
    F = F[np.sort(np.random.default_rng(n).permutation(F.shape[0])[:n])]
    return V, F.astype(np.int32)


@pytest.mark.parametrize("n", [2047, 2048, 5120, 20480])
def test_streams(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F = _mesh(n)
    lo_V, lo_F = M.icosphere(2)
    t = [torch.as_tensor(np.ascontiguousarray(x)).cuda() for x in
         (V, F, M.vertex_normals(V, F), lo_V.astype(np.float32), lo_F.astype(np.int32),
          M.face_grid_atlas(lo_F.shape[0], 128))]
    uv = torch.as_tensor(M.face_grid_atlas(n, 256)).cuda()
    eyes = torch.tensor([[0.0, 0.0, 3.0], [2.0, 2.0, 1.0]], device="cuda")
    ws = torch.empty(B.workspace_size(V.shape[0], n, lo_V.shape[0], lo_F.shape[0], 128), dtype=torch.uint8,
                     device="cuda")
    mws = torch.empty(B.view_maps_workspace_size(V.shape[0], n, 256, 2, 64), dtype=torch.uint8, device="cuda")
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    print(f"[gpu] second stream n={n}", flush=True)
    got = []
    for k in (0, 0, 0, 1, 0, 1, 1):
        with torch.cuda.stream(streams[k]):
            ws.fill_(255)
            mws.fill_(255)
            r = B.bake_normals(*t, 128, 0.3, workspace=ws)
            out = [r.map, r.hit]
            m = B.view_maps(t[0], t[1], uv, 256, eyes, (0, 0, 0), 0.5, 64, 5.0, 2e-3, workspace=mws)
            out += [m.uv, m.inc]
        torch.cuda.synchronize()
        assert r.status() == 0
        got.append([x.cpu().numpy() for x in out])
    for g in got[1:]:
        assert all(x.tobytes() == y.tobytes() for x, y in zip(got[0], g))
    b = B.BakeBatch([(*t, 128, 0.3)])
    b.forward()
    graph = b.capture()
    for _ in range(3):
        b.maps[0].zero_()
        b.workspace.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        assert b.maps[0].cpu().numpy().tobytes() == got[0][0].tobytes()
        assert b.hits[0].cpu().numpy().tobytes() == got[0][1].tobytes()


@pytest.mark.parametrize("n", [5120, 20480])
def test_eager_beside_a_capture(n):
    """A capture that forked into the second stream keeps it until it ends: bakes on
    another stream meanwhile run without it."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F = _mesh(n)
    lo_V, lo_F = M.icosphere(2)
    t = [torch.as_tensor(np.ascontiguousarray(x)).cuda() for x in
         (V, F, M.vertex_normals(V, F), lo_V.astype(np.float32), lo_F.astype(np.int32),
          M.face_grid_atlas(lo_F.shape[0], 128))]
    a, b = B.BakeBatch([(*t, 128, 0.3)]), B.BakeBatch([(*t, 128, 0.3)])
    other = torch.cuda.Stream()
    for _ in range(2):
        a.forward()
        b.forward(stream=other)
        b.forward(stream=other)
    torch.cuda.synchronize()
    want = a.maps[0].cpu().numpy()
    print(f"[gpu] eager beside a capture n={n}", flush=True)
    b.maps[0].zero_()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        a.forward()
        b.forward(stream=other)
        b.forward(stream=other)
        a.forward()
    torch.cuda.synchronize()
    assert b.maps[0].cpu().numpy().tobytes() == want.tobytes()
    for _ in range(2):
        a.maps[0].zero_()
        graph.replay()
        b.forward()
        torch.cuda.synchronize()
        assert a.maps[0].cpu().numpy().tobytes() == want.tobytes()

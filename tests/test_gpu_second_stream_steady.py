"""Bakes and view maps of few faces from one stream until they take the device's
second stream (after 16 calls), then from two threads with a stream each: the same
bits every time, with the workspace poisoned in between."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from test_gpu_second_stream import _mesh  # noqa: E402
from synth import meshes as M  # noqa: E402


@pytest.mark.parametrize("n", [2048, 20480])
def test_same_bits(n):
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
    torch.cuda.synchronize()
    print(f"[gpu] second stream steady n={n}", flush=True)

    def calls(stream, times, got):
        torch.cuda.set_device(0)
        with torch.cuda.stream(stream):
            ws = torch.empty(B.workspace_size(V.shape[0], n, lo_V.shape[0], lo_F.shape[0], 128), dtype=torch.uint8,
                             device="cuda")
            mws = torch.empty(B.view_maps_workspace_size(V.shape[0], n, 256, 2, 64), dtype=torch.uint8, device="cuda")
            for _ in range(times):
                ws.fill_(255)
                mws.fill_(255)
                r = B.bake_normals(*t, 128, 0.3, workspace=ws)
                m = B.view_maps(t[0], t[1], uv, 256, eyes, (0, 0, 0), 0.5, 64, 5.0, 2e-3, workspace=mws)
                got.append([r.map, r.hit, m.uv, m.inc])
            stream.synchronize()

    one, two, three = [], [], []
    calls(torch.cuda.Stream(), 24, one)  # from the ninth pair on with the second stream
    th = [threading.Thread(target=calls, args=(torch.cuda.Stream(), 24, g)) for g in (two, three)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    torch.cuda.synchronize()
    assert len(one) == len(two) == len(three) == 24
    want = [x.cpu().numpy().tobytes() for x in one[0]]
    for g in one + two + three:
        assert [x.cpu().numpy().tobytes() for x in g] == want

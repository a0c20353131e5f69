"""Simplification on both sides of the 2,560 faces up to which one workgroup finds
the rank of a round, with the most edges that it meets and with none that is
allowed.  Bit for bit the FP64 oracle's."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from test_gpu_qem_poles import edges_of_one_face, poles  # noqa: E402
from test_gpu_qem_valence import soup  # noqa: E402

CASES = [("2,560 faces", poles(40, 1, 2, 32)), ("2,562 faces", poles(61, 2, 2, 21)), ("7,680 edges", soup(2560, 3)),
         ("7,683 edges", soup(2561, 4)), ("none allowed", edges_of_one_face(30, 5)), ("one face", soup(1, 6))]


@pytest.mark.parametrize("rho", [0.01, 0.25, 1.0])
@pytest.mark.parametrize("name,mesh", CASES, ids=[c[0] for c in CASES])
def test_equals_the_oracle(oracle_lib, name, mesh, rho):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2605_26137_amd.bake as B
    V, F = mesh[0].astype(np.float32), np.ascontiguousarray(mesh[1].astype(np.int32))
    print(f"[gpu] qem small {name} rho={rho}", flush=True)
    Vd, Fd = torch.from_numpy(V).cuda(), torch.from_numpy(F).cuda()
    for target, rounds in ((4, 2), (max(4, F.shape[0] // 2), 1000)):
        r = B.qem_simplify(Vd, Fd, target, rho=rho, max_rounds=rounds)
        w = oracle_lib.qem_simplify(V, F, target, method="rounds", rho=rho, max_rounds=rounds)
        assert r.rounds == w.rounds, (target, rounds)
        np.testing.assert_array_equal(r.F.cpu().numpy(), w.F)
        np.testing.assert_array_equal(r.V.cpu().numpy(), w.V.astype(np.float32))

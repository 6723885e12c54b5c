"""ssp_rng_normals gives the normals that the FP64 step adds, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# few wavefronts: drawing waves; without the queue: the plain kernel; two beads a lane
@pytest.mark.parametrize("queue", [True, False])
@pytest.mark.parametrize("n", [5, 40, 100])
def test_rng_normals_are_the_steps(n, queue):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_2899_amd.ensemble import Ensemble
    # 2 dt = 2^-10: the step's scale is a power of two, so nothing is rounded differently
    e = Ensemble(n, 3, chain_ids=[7, 11, 500], precision="fp64", dt=2.0 ** -11, seed=9, corr_levels=0).init()
    e.set_schedule(queue)
    zero = torch.zeros((3 * n, 3), dtype=torch.float64, device=e.device)
    empty = torch.full((3 * n,), -1, dtype=torch.int32, device=e.device)
    for step in range(6):
        e.write_state(zero, zero, empty)  # no bonds and no springs: the move is the noise alone
        e.step(1)
        R = e.state()[0].cpu().numpy().reshape(3, n, 3)
        for k, gid in enumerate((7, 11, 500)):
            want = e.rng_normals(gid, step, 0, n).cpu().numpy()
            assert np.array_equal(R[k] * 2.0 ** 5, want), (step, gid)
    e.close()

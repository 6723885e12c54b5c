"""FP64 hops of finite states whose energy differences overflow to inf - inf: either
probability is 1/2, so that every spring away from the ends hops at every step."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# drawing waves, the plain kernel, and enough wavefronts for the queue; two beads a lane
@pytest.mark.parametrize("m,queue", [(3, True), (3, False), (2400, True)])
@pytest.mark.parametrize("n", [10, 80])
def test_springs_hop_when_the_energy_is_not_a_number(n, m, queue):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_2899_amd.ensemble import Ensemble
    e = Ensemble(n, m, precision="fp64", seed=9, corr_levels=0).init()
    e.set_schedule(queue)
    # offsets d of 1.2e308 with mixed signs, whose double overflows, on every bead, so
    # that all move alike and keep their bonds: b . (b + 2 d) = inf - inf + inf
    far = 6e307 * np.array([1.0, -1.0, 1.0])
    R = far + np.arange(n)[:, None] * np.full(3, 1e300)
    A = np.tile(-far, (n, 1))
    S = np.arange(n, dtype=np.int32)
    dev = lambda x, t: torch.tensor(np.tile(x, (m,) + (1,) * (x.ndim - 1)), dtype=t, device=e.device)
    e.write_state(dev(R, torch.float64), dev(A, torch.float64), dev(S, torch.int32))
    e.step(1)
    R1, _, got = (x.cpu().numpy() for x in e.state())
    assert np.isfinite(R1).all()
    got = got.reshape(m, n)
    inner = (S > 0) & (S < n - 1)
    moved = got[:, inner] - S[inner]
    kept = got[:, inner] >= 0  # (one hopped on to an end may be destroyed in the same step)
    assert np.all(np.abs(moved[kept]) == 1)
    assert (moved[kept] == 1).any() and (moved[kept] == -1).any()
    e.close()

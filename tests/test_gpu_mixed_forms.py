"""Groups of one launch in different step forms side by side (low-latency two-bead
groups beside queues, all low-latency with a common share, a group beyond its limit
beside a small one) against plain launches, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,chains", [
    ("fp32", {16: 6000, 32: 1400, 128: 90}), ("fp32", {16: 1100, 32: 1100, 64: 520}), ("fp32", {64: 1000, 128: 400}),
    ("fp32", {32: 4200, 64: 100}), ("fp64", {32: 420, 64: 100, 128: 450}), ("fp64", {8: 1300, 16: 900, 100: 40})])
def test_forms_side_by_side(precision, chains):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_2899_amd.ensemble import Ensemble
    N = np.concatenate([np.full(m, n, dtype=np.int32) for n, m in chains.items()])
    kap = np.zeros((1, 9))
    kap[0, 1] = 0.3
    out = []
    for queue in (True, False):
        e = Ensemble(N, precision=precision, seed=3, corr_levels=0, sample_every=5, series_capacity=20).init()
        e.set_schedule(queue)
        e.step(41, kap)
        e.step(20)
        out.append([x.cpu() for x in e.state()] + [e.element_series().cpu()])
        e.close()
    for a, b in zip(out[0][:3], out[1][:3]):
        assert torch.equal(a, b)
    s0, s1 = out[0][3], out[1][3]
    # sums of at most N squares of the same terms in another order, then over the chains
    assert torch.all((s0 - s1).abs() <= 200 * 2.3e-16 * s1.abs().max())

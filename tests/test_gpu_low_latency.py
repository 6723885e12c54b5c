"""The low-latency form of the step (drawing waves beside the stepping wave)
against one wavefront per task (ssp_set_schedule off), which the parity tests
hold to the oracle: bit for bit, for launches that start and end at every phase
of a step pair, both construction rules, at rest and under flow, and on either
side of the wave-task count where the queue takes over."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _run(N, M, calls, persistent, kap, **kw):
    from paper_1106_2899_amd.ensemble import Ensemble
    e = Ensemble(N, M, seed=13, sample_every=3, corr_levels=4, corr_batches=1, series_capacity=200, **kw)
    e.set_schedule(persistent)
    e.init()
    for n in calls:
        e.step(n, kap)
    out = [*e.state(), e.stress(), e.element_series(), torch.as_tensor(e.correlator()["G"])]
    e.close()
    return out


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("N,M,rule,rate", [(2, 70, 0, 0.0), (8, 64, 1, 0.0), (16, 5, 0, 0.3), (20, 33, 1, 0.1),
                                           (32, 64, 0, 0.0), (50, 7, 0, 0.2), (64, 3, 1, 0.0), (100, 4, 0, 0.1),
                                           (128, 3, 1, 0.0)])
def test_low_latency_form_equals_plain_launches_bitwise(N, M, rule, rate, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    kap = None if rate == 0.0 else np.array([0, rate, 0, 0, 0, 0, 0, 0, 0.0])
    calls = (1, 1, 2, 3, 5, 64, 1, 51)
    a, b = (_run(N, M, calls, p, kap, precision=precision, construct_rule=rule) for p in (True, False))
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("precision,N,M", [("fp32", 60, 2048), ("fp32", 60, 2049), ("fp32", 70, 1280), ("fp32", 70, 1281),
                                           ("fp64", 40, 512), ("fp64", 40, 513), ("fp64", 40, 1024),
                                           ("fp64", 40, 1025), ("fp64", 70, 512), ("fp64", 70, 513)])
def test_low_latency_form_at_its_limit(precision, N, M):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    a, b = (_run(N, M, (7, 30), p, None, precision=precision) for p in (True, False))
    for x, y in zip(a, b):
        assert torch.equal(x, y)

"""Step kernels of several mapping groups run on streams of their own: the same
as one group at a time (every group in an ensemble of its own), eagerly, from the
library's graph, and captured by the caller into a graph that is replayed."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LENGTHS = [8, 100, 16, 30, 64, 2, 128, 33, 17, 9]


@pytest.mark.parametrize("how", ["eager", "graph", "captured"])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_groups_on_streams_step_like_groups_apart(precision, how):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_2899_amd.ensemble import Ensemble
    N = np.resize(LENGTHS, 120).astype(np.int32)
    kap = np.array([0, 0.1, 0, 0, 0, 0, 0, 0, 0.0])
    steps, calls = 23, 4
    e = Ensemble(N, precision=precision, seed=6, sample_every=5, corr_levels=4, corr_batches=2, use_graph=how == "graph",
                 max_steps_per_launch=9)
    e.init()
    k = e.kappa_tensor(kap)
    if how == "captured":
        s = torch.cuda.Stream()
        e.stream = s
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            e.step(steps, k)
        e.stream = torch.cuda.current_stream()
    for _ in range(calls):
        if how == "captured":
            g.replay()
        else:
            e.step(steps, k)
        torch.cuda.synchronize()
        torch.ones(1000, device="cuda").sum().item()  # other work between the replays
    R, A, S = (x.cpu().numpy() for x in e.state())
    stress = e.stress().cpu().numpy()
    for lo, hi in ((2, 8), (9, 16), (17, 32), (33, 64), (65, 128)):
        ids = np.nonzero((N >= lo) & (N <= hi))[0]
        one = Ensemble(N[ids], chain_ids=ids, precision=precision, seed=6, corr_levels=0).init()
        one.step(steps * calls, kap)
        r, a, s1 = (x.cpu().numpy() for x in one.state())
        at = np.concatenate([np.arange(e.offsets[i], e.offsets[i] + N[i]) for i in ids])
        assert np.array_equal(s1, S[at]) and np.array_equal(r, R[at])
        occ = s1 >= 0
        assert np.array_equal(a[occ], A[at][occ])
        assert np.allclose(one.stress().cpu().numpy(), stress[ids], rtol=1e-13, atol=1e-11)
        one.close()
    e.close()

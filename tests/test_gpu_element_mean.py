"""The per-chain stress and its element means at the edges of their lane segments
(chains of 2..128 beads), of the blocks' rounds and of the split of an element
over several blocks: against numpy on the state read back."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _stress(R, A, S, ns):
    """sigma, sigma^v of one chain and the sums of the terms' magnitudes."""
    b = R[1:] - R[:-1]
    occ = S >= 0
    d = R[S[occ]] - A[occ]
    out, size = [], []
    for v, f, less in ((b, 3.0, len(R)), (d, 3.0 / ns, occ.sum())):
        for p, q in ((0, 0), (1, 1), (2, 2), (0, 1), (1, 2), (2, 0)):
            x = f * v[:, p] * v[:, q]
            out.append(x.sum() - (less if p == q else 0))
            size.append(np.abs(x).sum() + (less if p == q else 0))
    return np.array(out), np.array(size)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("lengths,sizes", [
    ([2, 15, 16], [1, 2, 60]), ([16], [1, 1, 64, 65]), ([17, 32, 2], [300, 7]), ([33, 64, 63], [33]),
    ([65, 128, 127, 3], [5, 40]), ([8], [1500]), ([20], [337, 336, 1]), ([40], [129])])
def test_stress_and_element_means(lengths, sizes, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_2899_amd.ensemble import Ensemble
    M = sum(sizes)
    N = np.resize(lengths, M).astype(np.int32)
    off = np.concatenate([[0], np.cumsum(sizes)])
    e = Ensemble(N, n_elements=len(sizes), element_offsets=off, precision=precision, seed=4, corr_levels=0).init()
    e.step(5)
    R, A, S = (x.cpu().numpy() for x in e.state())
    got, mean = e.stress().cpu().numpy(), e.element_stress().cpu().numpy()
    for k in range(M):
        o = e.offsets[k]
        want, size = _stress(R[o:o + N[k]], A[o:o + N[k]], S[o:o + N[k]], e.ns)
        # FP64 sums of at most N terms in another order, products rounded once
        assert np.all(np.abs(got[k] - want) <= (N[k] + 8) * 2.3e-16 * (size + 1.0)), k
    for i, n in enumerate(sizes):
        part = got[off[i]:off[i + 1]]
        want = np.array([math.fsum(part[:, c]) for c in range(12)]) / n
        assert np.all(np.abs(mean[i] - want) <= 8 * 2.3e-16 * np.abs(part).sum(0) / n)
    e.close()


def test_write_state_names_the_first_bad_chain():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_2899_amd._lib import SspError
    from paper_1106_2899_amd.ensemble import Ensemble
    N = np.resize([3, 16, 17, 40, 128], 500).astype(np.int32)
    e = Ensemble(N, precision="fp32", seed=4, corr_levels=0).init()
    R, A, S = e.state()
    before = e.stress()
    for chains, value in (([0], -2), ([499, 17], None), ([250], 1 << 30)):
        bad = S.clone()
        for c in chains:
            bad[int(e.offsets[c]) + int(N[c]) - 1] = int(N[c]) if value is None else value
        with pytest.raises(SspError, match=f"chain {min(chains)}$"):
            e.write_state(R, A, bad)
        assert torch.equal(e.stress(), before)
    e.write_state(R, A, S)
    assert torch.equal(e.stress(), before)
    e.close()

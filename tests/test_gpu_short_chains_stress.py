"""Chain stress and element means of ensembles whose mean length names a narrower
lane segment than their longest chain needs: segments of 4, 8, 16 and 32 lanes, long
chains in rounds of them, against numpy on the state read back."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _stress(R, A, S, ns):
    """sigma, sigma^v of one chain and the sums of the terms' magnitudes."""
    occ = S >= 0
    out, size = [], []
    for v, f, less in ((R[1:] - R[:-1], 3.0, len(R)), (R[S[occ]] - A[occ], 3.0 / ns, occ.sum())):
        for p, q in ((0, 0), (1, 1), (2, 2), (0, 1), (1, 2), (2, 0)):
            x = f * v[:, p] * v[:, q]
            out.append(x.sum() - (less if p == q else 0))
            size.append(np.abs(x).sum() + (less if p == q else 0))
    return np.array(out), np.array(size)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("short,long,sizes", [
    ([2, 3, 4], [], [1, 130, 7]), ([4], [128], [700]), ([3], [5, 9, 64], [66, 600]), ([5, 8], [17], [40, 1, 39]),
    ([8], [128, 127], [1030]), ([16], [33, 65], [500, 3]), ([24, 30], [128, 66], [90])])
def test_segments_narrower_than_the_longest_chain(short, long, sizes, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_2899_amd.ensemble import Ensemble
    M = sum(sizes)
    N = np.resize(short, M).astype(np.int32)
    for i, n in enumerate(long):
        N[(i + 1) * M // (len(long) + 1)] = n
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

"""The element series' sums over chains, at the edges of its rounds of lanes and
in both splits (one or four wavefronts per element and sample): against the
exactly rounded sums of the same ensemble's one-chain elements."""
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[1, 20, 21, 22, 3], [84, 85, 90], [1, 500], [83], [84], [337, 335, 336], [63, 64, 105]])
def test_series_sums_every_chain_of_its_element(sizes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_2899_amd.ensemble import Ensemble
    M, every, calls = sum(sizes), 3, (7, 11, 4)  # launches that start at different phases of the sampling
    cap = sum(calls) // every
    off = np.concatenate([[0], np.cumsum(sizes)])

    def series(offsets):
        e = Ensemble(6, M, n_elements=len(offsets) - 1, element_offsets=offsets, precision="fp64", seed=9,
                     sample_every=every, corr_levels=0, series_capacity=cap).init()
        for n in calls:
            e.step(n)
        s = e.element_series().cpu().numpy()
        e.close()
        return s

    one, got = series(np.arange(M + 1)), series(off)
    assert got.shape == (len(sizes), cap, 6)
    for e in range(len(sizes)):
        part = one[off[e]:off[e + 1]]
        for t in range(cap):
            for c in range(6):
                want, size = math.fsum(part[:, t, c]), np.abs(part[:, t, c]).sum()
                # compensated sums: the final rounding and a few of second order
                assert abs(got[e, t, c] - want) <= 4 * 2.2e-16 * size, (e, t, c)

"""The straight-line flow code (kappa with the xy entry alone, or the diagonal
alone, in a wavefront) against the general one: a chain steps the same, bit for
bit, whatever kappa the other chains of its wavefront have, and the general
code is held to the oracle by the parity tests."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

KAPPAS = [
    {1: 0.4},                               # simple shear
    {0: 0.05, 4: -0.025, 8: -0.025},        # uniaxial elongation
    {0: -0.04, 4: -0.02},                   # a diagonal without a positive entry
    {},                                     # at rest
    {0: 0.03, 1: 0.1, 5: -0.2, 6: 0.01},    # no special shape
    {1: -0.02},
    {8: 0.06},
]


def _kappa(d):
    k = np.zeros(9)
    for q, v in d.items():
        k[q] = v
    return k


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("N", [5, 16, 20, 33, 100])
def test_flow_shapes_step_like_the_general_code(N, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_2899_amd.ensemble import Ensemble
    M, steps = 2 * len(KAPPAS), 151
    kap = np.stack([_kappa(KAPPAS[i % len(KAPPAS)]) for i in range(M)])
    e = Ensemble(N, M, n_elements=M, element_offsets=np.arange(M + 1), precision=precision, seed=3, corr_levels=0)
    e.init().step(steps, kap)
    R, A, S = (x.cpu().numpy().reshape(M, N, -1) for x in e.state())
    e.close()
    for i in range(len(KAPPAS)):
        ids = [i, i + len(KAPPAS)]
        one = Ensemble(N, 2, precision=precision, seed=3, corr_levels=0, chain_ids=ids)
        one.init().step(steps, kap[i])
        r, a, s = (x.cpu().numpy().reshape(2, N, -1) for x in one.state())
        one.close()
        assert np.array_equal(s, S[ids]), KAPPAS[i]
        assert np.array_equal(r, R[ids]), KAPPAS[i]
        occ = s[..., 0] >= 0
        assert np.array_equal(a[occ], A[ids][occ]), KAPPAS[i]

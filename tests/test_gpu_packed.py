"""Plain steps with chains packed side by side in a wavefront against one chain
per lane segment (ssp_set_schedule off), which the parity tests hold to the
oracle: states bit for bit, sums of the stress to rounding.  Ensembles just large
enough to be packed, with chains that fill a wavefront, leave a remainder, take
fewer lanes than the twelve stress values, and, with two beads per lane, odd
lengths; elements of one chain and of many; every shape of flow."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("lo,hi,M,E,rule,flow", [
    (16, 128, 3300, 40, 0, True), (2, 64, 6000, 7, 1, True), (20, 20, 5300, 3, 0, False), (2, 5, 40000, 5, 1, False),
    (9, 11, 21000, 300, 0, True), (65, 128, 3000, 1500, 0, True), (2, 128, 4200, 1, 1, False)])
def test_packed_chains_step_like_segments(lo, hi, M, E, rule, flow, precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_2899_amd.ensemble import Ensemble
    rng = np.random.default_rng(M)
    N = rng.integers(lo, hi + 1, size=M).astype(np.int32)
    kap = None
    if flow:
        kap = np.zeros((E, 9))
        kind = np.arange(E) % 4
        kap[kind == 0, 1] = 0.1
        kap[kind == 1] = np.array([0.05, 0, 0, 0, -0.025, 0, 0, 0, -0.025])
        kap[kind == 2] = 0.05 * rng.normal(size=9)
    out = []
    for packed in (True, False):
        e = Ensemble(N, n_elements=E, precision=precision, seed=3, sample_every=3, corr_levels=4, corr_batches=1,
                     series_capacity=30, construct_rule=rule)
        e.set_schedule(packed)
        e.init()
        for n in (1, 6, 33):
            e.step(n, kap)
        out.append([*e.state(), e.stress(), e.element_series(), torch.as_tensor(e.correlator()["G"])])
        e.close()
    (R, A, S, stress, series, G), (r, a, s, stress1, series1, G1) = out
    assert torch.equal(S, s) and torch.equal(R, r) and torch.equal(stress, stress1)
    occ = S >= 0
    assert torch.equal(A[occ], a[occ])
    # FP64 sums of at most 128 terms a chain in another order
    assert (series - series1).abs().max() <= 1e-13 * series1.abs().max()
    assert (G - G1).abs().max() <= 1e-13 * G1.abs().max()


@pytest.mark.parametrize("mapping", [None, [(9, 16, 16, 1), (17, 32, 32, 1), (33, 64, 64, 1)], [(9, 64, 64, 1)]])
def test_packed_chains_with_mappings_set(mapping):
    """The default mapping set again (which leaves the chains packed) and another
    one, against segments, at rest."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_2899_amd.ensemble import Ensemble
    N = np.random.default_rng(1).integers(9, 65, size=6000).astype(np.int32)
    out = []
    for packed in (True, False):
        e = Ensemble(N, n_elements=3, precision="fp32", seed=3, sample_every=5, corr_levels=0)
        e.set_schedule(packed)
        e.init()
        e.step(4)
        for m in mapping or []:
            e.set_mapping(*m)
        e.step(21)
        out.append([*e.state(), e.stress()])
        e.close()
    (R, A, S, stress), (r, a, s, stress1) = out
    occ = S >= 0
    assert torch.equal(S, s) and torch.equal(R, r) and torch.equal(A[occ], a[occ])
    # FP64 sums of at most 64 beads' terms, in an order that may depend on the mapping
    assert (stress - stress1).abs().max() <= 1e-13 * stress1.abs().max()

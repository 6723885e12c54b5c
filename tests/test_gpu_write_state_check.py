"""ssp_write_state refuses slots outside their chain on both sides of the number of
slots up to which the host checks them, names the first bad chain and writes nothing."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("last", [2, 3])  # 16384 slots, 16385
def test_write_state_check_on_both_sides(last):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_2899_amd._lib import SspError
    from paper_1106_2899_amd.ensemble import Ensemble
    N = np.full(8192, 2, dtype=np.int32)
    N[-1] = last
    e = Ensemble(N, precision="fp32", seed=4, corr_levels=0).init()
    R, A, S = (x.clone() for x in e.state())
    off = np.concatenate([[0], np.cumsum(N)])
    for chains in ([0], [8191], [4000, 17], [8190, 8191]):
        for value in (-2, 3):
            bad = S.clone()
            for c in chains:
                bad[int(off[c + 1]) - 1] = value
            with pytest.raises(SspError, match=f"chain {min(chains)}$"):
                e.write_state(R + 1.0, A, bad)
    assert torch.equal(e.state()[0], R)
    full = torch.tensor(np.concatenate([np.arange(n) for n in N]).astype(np.int32), device=e.device)
    e.write_state(R, A, full)  # the largest value a slot may have
    assert torch.equal(e.state()[2], full)
    e.close()

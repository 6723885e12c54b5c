"""The element means of the gradients and of the stress go through one scratch area
of the handle: a call that used it has ended on the device when it returns, so that
the next may come on another stream."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("ckpt", [4, 8])  # replayed segments, a stored window
def test_gradient_means_are_done_on_return(noalloc, ckpt):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import ctypes

    from paper_1106_2899_amd._lib import lib
    from paper_1106_2899_amd.ensemble import Ensemble
    M, E = 20000, 2  # parts of an element: from 337 chains on
    kap = np.zeros((E, 9))
    kap[:, 1] = [0.2, 0.4]
    e = Ensemble(12, M, n_elements=E, seed=6, corr_levels=0).init()
    e.forward_record(8, ckpt, kap)
    want_g, chain = e.adjoint_elements(3)
    want_s = e.element_stress()
    torch.cuda.synchronize()
    assert torch.allclose(want_g, chain.reshape(E, M // E, 10).mean(1), rtol=1e-11, atol=1e-11)
    assert torch.allclose(want_s, e.stress().reshape(E, M // E, 12).mean(1), rtol=1e-11, atol=1e-11)
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    got = torch.zeros_like(want_g)
    torch.cuda.synchronize()
    for _ in range(20):
        e.stream = one
        if noalloc:
            rc = lib().ssp_adjoint_elements_noalloc(e._h, ctypes.c_void_p(e._rec_p), e._rec_kappa_p, 3, 1,
                                                    ctypes.c_void_p(got.data_ptr()), e._s)
        else:
            rc = lib().ssp_adjoint_elements(e._h, ctypes.c_void_p(e._rec_p), e._rec_kappa_p, 3, 1,
                                            ctypes.c_void_p(chain.data_ptr()), ctypes.c_void_p(got.data_ptr()), e._s)
        done = one.query()
        e.stream = two
        s = e.element_stress()
        assert rc == 0 and done
        torch.cuda.synchronize()
        assert torch.equal(s, want_s) and torch.equal(got, want_g)
    e.close()


@pytest.mark.parametrize("ckpt", [4, 8])
def test_no_gradient_is_written_from_a_changed_recording(ckpt):
    """The means are queued before the error flags are read: on an error they leave
    the output as it was."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import ctypes

    from paper_1106_2899_amd._lib import lib
    from paper_1106_2899_amd.ensemble import Ensemble
    N, M, E, T = 12, 1000, 2, 8
    kap = np.zeros((E, 9))
    kap[:, 1] = [0.2, 0.4]
    e = Ensemble(N, M, n_elements=E, seed=6, corr_levels=0).init()
    e.forward_record(T, ckpt, kap)
    off = e._rec_p - e._rec_t.data_ptr()
    e._rec_t[off:off + (T + 1) * N * M].view(T + 1, N * M)[5, 3] = 100  # no such bead: read as an empty slot
    got = torch.full((E, 10), 7.5, dtype=torch.float64, device=e.device)
    chain = torch.zeros((M, 10), dtype=torch.float64, device=e.device)
    torch.cuda.synchronize()
    out, s = ctypes.c_void_p(got.data_ptr()), e._s
    rc = lib().ssp_adjoint_elements(e._h, ctypes.c_void_p(e._rec_p), e._rec_kappa_p, 3, 1,
                                    ctypes.c_void_p(chain.data_ptr()), out, s)
    rc2 = lib().ssp_adjoint_elements_noalloc(e._h, ctypes.c_void_p(e._rec_p), e._rec_kappa_p, 3, 1, out, s)
    torch.cuda.synchronize()
    assert rc != 0 and rc2 != 0
    assert (got == 7.5).all()
    e.close()

"""What a call whose solves do not all converge leaves behind: the direct
solver's solutions of the orbitals that did, bit for bit."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _poisson(torch, rho, n, h, tol, max_iter, precision):
    """Status, potentials, iterations and residuals of the C entry point."""
    from paper_2108_01186_amd import fsic as F
    t = torch.tensor(rho, device="cuda")
    v = torch.empty_like(t)
    g = F.make_grid(n, h, [-h * (m - 1) / 2 for m in n])
    it = (ctypes.c_int32 * len(rho))()
    rr = (ctypes.c_double * len(rho))()
    st = F.fsic_op_poisson(ctypes.byref(g), 12, 6, len(rho), ctypes.c_void_p(t.data_ptr()), ctypes.c_void_p(v.data_ptr()),
                           tol, max_iter, precision, F.FSIC_PCG, it, rr,
                           ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    return st, v.cpu().numpy(), np.array(it), np.array(rr)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_nonfinite_density_among_good_ones(torch_cuda, precision, value):
    """One bad density: the call reports it, with max_iter iterations, and the
    others' potentials, iterations and residuals are those of a call without it."""
    from paper_2108_01186_amd import fsic as F
    print(f"direct solver with a density of {value}, precision {precision}", flush=True)
    n, h = (24, 22, 20), 0.3
    rho = np.random.default_rng(3).random((5, n[0] * n[1] * n[2]))
    st, good, it, rr = _poisson(torch_cuda, rho, n, h, 1e-11, 5000, precision)
    assert st == 0
    rho[2, 777] = value
    st, v, itb, rrb = _poisson(torch_cuda, rho, n, h, 1e-11, 5000, precision)
    assert st == F.FSIC_ENOCONV
    for k in (0, 1, 3, 4):
        assert np.array_equal(v[k], good[k]) and itb[k] == it[k] and rrb[k] == rr[k], k
    assert itb[2] == 5000


@pytest.mark.parametrize("precision", [0, 1])
def test_iteration_limit_keeps_the_solution(torch_cuda, precision):
    """A tolerance that one application does not meet with no further iteration
    allowed: the potentials are those of that application."""
    from paper_2108_01186_amd import fsic as F
    print(f"direct solver at its iteration limit, precision {precision}", flush=True)
    n, h = (40, 37, 33), 0.3
    rho = np.random.default_rng(4).random((3, n[0] * n[1] * n[2]))
    st, good, it, rr = _poisson(torch_cuda, rho, n, h, 1e-11, 100, precision)
    assert st == 0 and np.all(it == 1)
    st, v, itb, rrb = _poisson(torch_cuda, rho, n, h, 1e-16, 1, precision)
    assert st == F.FSIC_ENOCONV
    assert np.array_equal(v, good) and np.array_equal(rrb, rr) and np.all(itb == 1)
    # two more applications meet it
    st, v, itb, rrb = _poisson(torch_cuda, rho, n, h, 1e-16, 100, precision)
    assert st == 0 and np.all(itb >= 2) and np.all(itb <= 3)

"""The work memory that context-free calls keep is given back on request, also
while calls run in other threads."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _poisson(F, rho, n, h):
    return F.op_poisson(rho, (n, n, n), h, [-h * (n - 1) / 2] * 3, tol=1e-9, solver="pcg")[0]


def test_kept_memory_is_given_back(torch_cuda):
    """Eight 64^3 densities take two work fields of 16.8 MB at least."""
    from paper_2108_01186_amd import fsic as F
    torch = torch_cuda
    print("release workspace", flush=True)
    n = 64
    rho = torch.rand((8, n ** 3), dtype=torch.float64, device="cuda")
    _poisson(F, rho, n, 0.3)  # torch's buffers and the library's tables are there
    torch.cuda.synchronize()
    held = torch.cuda.mem_get_info()[0]
    F.release_workspace()
    free = torch.cuda.mem_get_info()[0]
    assert free - held >= 2 * 8 * n ** 3 * 8
    ref = _poisson(F, rho, n, 0.3).cpu().numpy()
    F.release_workspace()
    F.release_workspace()  # nothing kept
    assert torch.cuda.mem_get_info()[0] >= free - (4 << 20)
    assert np.array_equal(_poisson(F, rho, n, 0.3).cpu().numpy(), ref)


def test_release_while_calls_run(torch_cuda):
    from paper_2108_01186_amd import fsic as F
    torch = torch_cuda
    print("release workspace while calls run", flush=True)
    rho = {n: torch.rand((2, n ** 3), dtype=torch.float64, device="cuda") for n in (20, 24)}
    ref = {n: _poisson(F, rho[n], n, 0.3).cpu().numpy() for n in rho}
    torch.cuda.synchronize()
    err, left = [], [len(rho)]

    def work(n):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(20):
                    if not np.array_equal(_poisson(F, rho[n], n, 0.3).cpu().numpy(), ref[n]):
                        err.append(n)
        except Exception as e:  # noqa: BLE001
            err.append(e)
        finally:
            left[0] -= 1

    ts = [threading.Thread(target=work, args=(n,)) for n in rho]
    for t in ts:
        t.start()
    while left[0] > 0:
        F.release_workspace()
    for t in ts:
        t.join()
    assert not err, err

"""The blocks that context-free calls keep from one call for the next: what a
call leaves in them reaches no later result, whatever the sizes in between,
and threads on streams of their own do not share one."""
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


def _calls(torch, n, count, seed, bad=False):
    """Every context-free call that takes work memory, results on the host."""
    from paper_2108_01186_amd import fsic as F
    rng = np.random.default_rng(seed)
    M = n ** 3
    h, origin = 0.4, np.zeros(3)
    dev = lambda a: torch.tensor(a, device="cuda")
    out = []
    psi = np.linalg.qr(rng.standard_normal((M, count)))[0].T / h ** 1.5
    v = rng.standard_normal(M)
    rho = rng.random((count, M))
    S = psi @ psi.T * h ** 3 + 0.1 * np.eye(count)
    if bad:
        rho[:] = v[:] = np.nan
    out.append(F.op_hamiltonian(dev(psi), dev(v), (n, n, n), h))
    for kw in ({"solver": "pcg"}, {"solver": "cg", "precision": "fp64"}, {"solver": "aar", "precision": "fp64"}):
        try:
            out.append(F.op_poisson(dev(rho), (n, n, n), h, origin, tol=1e-9, max_iter=400, **kw)[0])
        except F.FsicError:
            assert bad
    out += list(F.op_flo(dev(psi), origin + h * (2.5 + (n - 6) * rng.random((count, 3))), (n, n, n), h, origin))
    out += list(F.op_invsqrt(dev(S)))
    return [o.cpu().numpy() for o in out]


def test_kept_blocks_carry_nothing_over(torch_cuda):
    torch = torch_cuda
    print("kept blocks", flush=True)
    first = {(n, c): _calls(torch, n, c, n) for n, c in ((20, 3), (27, 2))}
    _calls(torch, 20, 3, 1, bad=True)   # leaves NaN in blocks of the same sizes
    _calls(torch, 33, 5, 2, bad=True)   # and in larger ones
    for (n, c), ref in first.items():
        for a, b in zip(ref, _calls(torch, n, c, n)):
            assert np.array_equal(a, b)


def test_threads_on_their_own_streams(torch_cuda):
    torch = torch_cuda
    print("threads", flush=True)
    ref = {n: _calls(torch, n, 2, n) for n in (18, 20, 22, 24)}
    got, err = {}, []

    def work(n):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                got[n] = [_calls(torch, n, 2, n) for _ in range(3)]
        except Exception as e:  # noqa: BLE001
            err.append(e)

    ts = [threading.Thread(target=work, args=(n,)) for n in ref]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not err, err
    for n, runs in got.items():
        for run in runs:
            for a, b in zip(ref[n], run):
                assert np.array_equal(a, b)

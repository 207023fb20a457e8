"""The boundary bases a context keeps are bounded: those least recently used
go, none that the pass in hand needs, and a grid that comes back is solved
again with the same results."""
import numpy as np
import pytest

from paper_2108_01186_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def test_bases_are_bounded(torch_cuda, monkeypatch):
    """Basis of an n^3 grid at lmax 6: 2 x 49 octants of (n/2)^3 doubles, 3.2 MB
    at 32^3, 4.5 MB at 36^3, 6.3 MB at 40^3 (octants of 16, 18 and 20)."""
    from paper_2108_01186_amd import fsic as F
    torch = torch_cuda
    print("basis limit", flush=True)
    systems = {}
    for n in (32, 36, 40):
        s = synth.make_molecule("basis", n, 10.0 / (n - 1), 3, 8, (3,), seed=n)
        s.psi = [torch.as_tensor(np.ascontiguousarray(p), device="cuda") for p in s.psi]
        systems[n] = F.system_dict(s)
    ctx = F.Context(tol=1e-11, flags=F.FSIC_WANT_VSIC | F.FSIC_KEEP_TAPE)

    def step(*ns):
        e, U, X, g, st, _ = ctx.forward_backward([systems[n] for n in ns])
        ref = first.setdefault(ns, (e.copy(), [np.concatenate(s) for s in g]))
        # (a basis takes the transform layout of the pass that solves it: residual
        # 1e-13 times 4 n^2 / pi^2, below 700)
        assert np.abs(e - ref[0]).max() < 1e-10
        assert all(np.abs(np.concatenate(a) - b).max() < 1e-10 for a, b in zip(g, ref[1]))
        return st["basis_solves"] // 49

    first = {}
    # room for all
    assert [step(32), step(36), step(40), step(32), step(36), step(40)] == [1, 1, 1, 0, 0, 0]
    # room for 36^3 and 40^3 (10.8 MB) or 32^3 and 40^3 (9.5), not all three (14)
    monkeypatch.setenv("FSIC_BASIS_MB", "11")
    ctx.close()
    ctx = F.Context(tol=1e-11, flags=F.FSIC_WANT_VSIC | F.FSIC_KEEP_TAPE)
    assert [step(32), step(40), step(32)] == [1, 1, 0]
    assert step(36) == 1                 # 40^3 goes, the older
    assert [step(32), step(36)] == [0, 0]
    assert step(40) == 1                 # 32^3 goes
    assert [step(36), step(40)] == [0, 0]
    assert step(32, 36, 40) == 1         # one pass has all it needs
    assert step(32, 36, 40) == 0
    # none kept beyond the pass that uses it
    monkeypatch.setenv("FSIC_BASIS_MB", "0")
    assert [step(32), step(36), step(36), step(32)] == [0, 0, 0, 0]  # nothing new: nothing to make room for
    ctx.close()
    ctx = F.Context(tol=1e-11, flags=F.FSIC_WANT_VSIC | F.FSIC_KEEP_TAPE)
    assert [step(32), step(36), step(36), step(32)] == [1, 1, 0, 1]
    # a further backward pass on the tape whose bases are kept
    g = ctx.backward([[3]])
    assert np.abs(np.concatenate(g[0]) - first[(32,)][1][0]).max() < 1e-9
    ctx.close()

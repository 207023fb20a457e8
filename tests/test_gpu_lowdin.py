"""The N x N kernels (lowdin.hip) where their layout changes: pair counts that
fill a wave or not, odd N (a padded row), the step from one block a thread to
four and from LDS to scratch (N = 64, 65), and the largest channel."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
EPS = np.finfo(float).eps


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("N", [1, 2, 3, 4, 15, 17, 32, 33, 63, 64, 65, 66, 95, 127, 128])
@pytest.mark.parametrize("scale", [1.0, 1e-200])
def test_inverse_square_root(torch_cuda, N, scale):
    """Z S Z = 1 and the eigenvalues against LAPACK.  A sweep rotates every
    entry N times with about 6 roundings, ten sweeps at most are needed here:
    the computed factors are exact for S + E, |E| < 64 N eps |S|, which moves
    the eigenvalues by |E| and Z S Z by |E| over the smallest one.  Entries
    far below one must not underflow in the angles (their squares do)."""
    from paper_2108_01186_amd import fsic as F
    torch = torch_cuda
    print(f"invsqrt N={N} {scale}", flush=True)
    rng = np.random.default_rng(N)
    B = rng.standard_normal((N, N))
    S = B @ B.T / N + 0.05 * np.eye(N)
    w = np.linalg.eigvalsh(S)
    if scale != 1.0:
        # a well scaled block and entries whose squares underflow beside it
        k = N // 2
        S[:k, k:] *= scale
        S[k:, :k] *= scale
        w = np.linalg.eigvalsh(S)
    Z, lam = F.op_invsqrt(torch.tensor(S, device="cuda"))
    Z, lam = Z.cpu().numpy(), lam.cpu().numpy()
    assert np.abs(np.sort(lam) - w).max() <= 64 * N * EPS * w[-1]
    assert np.abs(Z @ S @ Z - np.eye(N)).max() <= 64 * N * EPS * w[-1] / w[0]


@pytest.mark.parametrize("N", [2, 15, 17, 33, 63, 65])
def test_gradient_along_a_direction(torch_cuda, N):
    """The reverse chain against central differences of the energy: halving
    the step leaves a quarter of the truncation error, so the difference of
    the two quotients bounds what is left in the finer one three times over;
    the energies carry the solver's tolerance."""
    from paper_2108_01186_amd import fsic as F, synth
    torch = torch_cuda
    print(f"gradient N={N}", flush=True)
    s = synth.make_molecule("lw", 22, 0.5, max(N, 3), int(2.4 * max(N, 3)) + 1, (N,), seed=90 + N, atom_box=7.0)
    psi = torch.as_tensor(np.ascontiguousarray(s.psi[0]), device="cuda")
    # away from the cells' faces, where the interpolant's derivative jumps
    cell = (s.fod[0] - s.origin) / s.h
    fod = s.origin + s.h * (np.floor(cell) + np.clip(cell - np.floor(cell), 0.1, 0.9))
    ctx = F.Context(tol=1e-12, flags=F.FSIC_KEEP_TAPE)
    sysd = lambda fod: {"n": s.n, "h": s.h, "origin": s.origin, "psi": [psi], "fod": [fod]}
    e, U, X, g, st, _ = ctx.forward_backward([sysd(fod)])
    d = np.random.default_rng(N).standard_normal((N, 3))
    d /= np.linalg.norm(d)
    energy = lambda t: float(ctx.forward([sysd(fod + t * d)])[0][0])
    step = 1e-3
    fine, coarse = [(energy(t) - energy(-t)) / (2 * t) for t in (step, 2 * step)]
    total = float(np.abs(np.concatenate([np.ravel(x) for x in U])).sum())
    assert abs((g[0][0] * d).sum() - fine) <= abs(fine - coarse) + 1e-11 * total / step
    ctx.close()

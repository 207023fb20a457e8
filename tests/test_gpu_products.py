"""The Gram matrix, the orbital transform and the adjoint contraction at the
orbital counts where their kernels change (register and LDS fragments, one or
four waves per tile set, partial tiles) and on grids of odd and even node
counts, against numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


SIZES = [1, 16, 17, 32, 33, 48, 49, 64, 65, 80, 96, 97, 112, 128]


@pytest.mark.parametrize("N", SIZES)
@pytest.mark.parametrize("n", [(11, 13, 9), (12, 10, 16)])
def test_gram(torch_cuda, N, n):
    """G of random orthonormalised rows against numpy's product (M products
    of size 1/M, summed in another order: M rounding errors at most)."""
    from paper_2108_01186_amd import fsic as F
    torch = torch_cuda
    print(f"gram N={N} {n}", flush=True)
    M = n[0] * n[1] * n[2]
    h = 0.5
    rng = np.random.default_rng(N + M)
    q = np.linalg.qr(rng.standard_normal((M, N)))[0].T
    psi = np.ascontiguousarray(q / np.sqrt(h ** 3))
    # FODs at distinct inner nodes' neighbourhoods
    cells = rng.permutation((n[0] - 4) * (n[1] - 4) * (n[2] - 4))[:N]
    ijk = np.stack([cells % (n[0] - 4), cells // (n[0] - 4) % (n[1] - 4), cells // ((n[0] - 4) * (n[1] - 4))], 1) + 1.5
    G = F.op_flo(torch.tensor(psi, device="cuda"), ijk * h, n, h, np.zeros(3))[1].cpu().numpy()
    assert np.abs(G - h ** 3 * psi @ psi.T).max() < M * np.finfo(float).eps


@pytest.mark.parametrize("N", SIZES)
@pytest.mark.parametrize("n", [(11, 13, 9), (12, 10, 16)])
def test_transform(torch_cuda, N, n):
    """Orbitals on disjoint node sets with each FOD on a node of its own
    orbital: T and S are diagonal, so every orbital is its psi times Z_ii T_ii
    (two roundings) and exactly zero on the others' nodes, which a misplaced
    row, node or contraction step would break."""
    from paper_2108_01186_amd import fsic as F
    torch = torch_cuda
    print(f"transform N={N} {n}", flush=True)
    M = n[0] * n[1] * n[2]
    h = 0.5
    rng = np.random.default_rng(N + M)
    inner = [(k * n[1] + j) * n[0] + i for k in range(1, n[2] - 2) for j in range(1, n[1] - 2) for i in range(1, n[0] - 2)]
    fod_node = rng.permutation(inner)[:N]
    owner = rng.integers(0, N, M)
    owner[fod_node] = np.arange(N)
    psi = np.zeros((N, M))
    psi[owner, np.arange(M)] = rng.uniform(0.5, 1.5, M)
    psi /= np.sqrt(h ** 3 * (psi ** 2).sum(1, keepdims=True))
    fod = h * np.stack([fod_node % n[0], fod_node // n[0] % n[1], fod_node // (n[0] * n[1])], 1)
    T, G, S, Z, phi = (x.cpu().numpy() for x in F.op_flo(torch.tensor(psi, device="cuda"), fod, n, h, np.zeros(3)))
    ref = (np.diag(Z) * np.diag(T))[:, None] * psi
    assert np.all(phi[ref == 0] == 0)
    assert np.abs(phi - ref).max() <= 4 * np.finfo(float).eps * np.abs(ref).max()


@pytest.mark.parametrize("nocc", [(1,), (16, 17), (33, 48), (49, 64), (65, 20)])
def test_contraction_in_the_gradient(torch_cuda, nocc):
    """The adjoint contraction of both channels of a system (in one launch per
    shape) through the FOD gradient, against the ghost-node path, whose source
    comes from another kernel but uses the same contraction, and against the
    gradient of each channel alone, whose blocks and sums differ."""
    from paper_2108_01186_amd import fsic as F, synth
    torch = torch_cuda
    print(f"contraction {nocc}", flush=True)
    N = max(nocc)
    s = synth.make_molecule("con", 22, 0.5, max(N, 3), int(2.4 * max(N, 3)) + 1, nocc, seed=70 + N, atom_box=7.0)
    psi = [torch.as_tensor(np.ascontiguousarray(p), device="cuda") for p in s.psi]

    def grad(chans):
        d = {"n": s.n, "h": s.h, "origin": s.origin, "psi": [psi[c] for c in chans], "fod": [s.fod[c] for c in chans]}
        ctx = F.Context(tol=1e-11, flags=F.FSIC_KEEP_TAPE)
        e, U, X, g, st, _ = ctx.forward_backward([d])
        ctx.close()
        return g[0], st["cond_S_max"]

    both, cond = grad(range(len(nocc)))
    for c in range(len(nocc)):
        one, _ = grad([c])
        # the sums' order moves S by rounding, which cond(S) carries into the gradient
        assert np.abs(both[c] - one[0]).max() < 1e-13 * max(cond, 1e2) * max(1.0, np.abs(one[0]).max()), c

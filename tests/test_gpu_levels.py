"""Small dense problems run through the offset-list kernels, everything in one block
(block tiles, wave tiles, elementwise sums of private copies), larger ones through
the GEMM kernels (FTCC_DENSE_LEVELS=0: always).  Both against each other at sizes
around the tile edges: one residual is a sum of at most n^3 products per element in
FP64, so the two orders of summation differ by a few times n^1.5 * 2^-53 of the
largest element (n = 40: 3e-14); 1e-12 is allowed."""
import numpy as np
import pytest

import ftcc_inputs as fi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2004_01729_amd import ftcc
    return ftcc


def _close(a, b, tol=1e-12):
    a, b = np.asarray(a), np.asarray(b)
    return np.abs(a - b).max() <= tol * max(np.abs(b).max(), 1e-3)


@pytest.mark.parametrize("n", [1, 2, 5, 8, 16, 17, 31, 33, 40])
def test_residual_both_paths(F, monkeypatch, n):
    h, eri, eps = fi.random_hamiltonian(n, seed=n, scale=0.1)
    t1, t2 = fi.random_amplitudes(n, seed=n + 1, scale=0.05)
    out = []
    for lev in (None, "0"):
        if lev:
            monkeypatch.setenv("FTCC_DENSE_LEVELS", lev)
        print(f"[levels] residual n={n} FTCC_DENSE_LEVELS={lev}", flush=True)
        ctx = F.Context(1, n_tau=6, nodes_per_panel=3)
        ctx.set_hamiltonian(0, h, eri, eps)
        out.append(ctx.eval_residual(0, 0.1, 2.0, t1, t2))
        ctx.close()
    for a, b in zip(*out):
        assert _close(a, b)


@pytest.mark.parametrize("spin", [False, True])
def test_step_both_paths(F, monkeypatch, spin):
    """A whole step of a batch of different sizes (restricted) and of a Neel
    reference (spin orbitals): Omega, Lambda and the derivatives."""
    if spin:
        systems = [fi.hubbard_unrestricted(L=4, U=2.0, T=1.0, reference="neel")]
    else:
        systems = [fi.hubbard_config(L=L, U=2.0, T=1.0) for L in (3, 17, 8)]
    out = []
    for lev in (None, "0"):
        if lev:
            monkeypatch.setenv("FTCC_DENSE_LEVELS", lev)
        print(f"[levels] step spin={spin} FTCC_DENSE_LEVELS={lev}", flush=True)
        ctx = F.Context(len(systems), n_tau=8, nodes_per_panel=4, tol=1e-13, spin_orbital=int(spin))
        for i, s in enumerate(systems):
            ctx.set_hamiltonian(i, s.h, s.eri, s.eps)
        ctx.solve([s.mu for s in systems], [s.beta for s in systems])
        om, parts = ctx.grand_potential()
        ctx.lam()
        lam = ctx.get_lambda(0, 2)
        r = ctx.response(want_mu=True, want_beta=True, want_h=True, want_eps=True)
        ctx.close()
        out.append([om, parts, *lam, r["mu"], r["beta"], *r["h"], *r["eps"]])
    for a, b in zip(*out):
        assert _close(a, b, 1e-11)   # the sweeps stop at 1e-13 of the amplitudes


@pytest.mark.parametrize("split", [(15, 15), (8, 14), (22, 11)])
def test_two_label_blocks(F, split):
    """Two labels (p + q + r + s even): blocks of unequal, odd sizes whose elements share
    the four-wide elementwise kernel's blocks, against the same problem without labels."""
    n = sum(split)
    lab = np.arange(n) % 2 if split[0] == split[1] else np.repeat([0, 1], split)
    h, eri, eps = fi.random_hamiltonian(n, seed=n, scale=0.1)
    t1, t2 = fi.random_amplitudes(n, seed=n + 1, scale=0.05)
    even2 = (lab[:, None] + lab[None, :]) % 2 == 0
    even4 = (lab[:, None, None, None] + lab[:, None, None] + lab[:, None] + lab) % 2 == 0
    h, t1, eri, t2 = h * even2, t1 * even2, eri * even4, t2 * even4
    out = []
    for labelled in (True, False):
        print(f"[levels] two labels {split} labelled={labelled}", flush=True)
        ctx = F.Context(1, n_tau=6, nodes_per_panel=3)
        ctx.set_hamiltonian(0, h, eri, eps)
        if labelled:
            ctx.set_momentum(0, lab, [2])
        out.append(ctx.eval_residual(0, 0.1, 2.0, t1, t2))
        ctx.close()
    for a, b in zip(*out):
        assert _close(a, b)


@pytest.mark.parametrize("L", [32, 33, 40])
def test_wide_wave_tiles(F, L):
    """Rings with a label per orbital: L blocks of L x L outputs over L inner indices, in
    32 x 32 wave tiles (whole ones, remainders of 1 and of 8), against the same ring
    without labels."""
    s = fi.hubbard_config(L=L, U=2.0, T=1.0)
    lab = np.arange(L)
    t1, t2 = fi.random_amplitudes(L, seed=L, scale=0.05)
    t1 = np.diag(np.diag(t1))
    t2 = t2 * ((lab[:, None, None, None] + lab[:, None, None] - lab[:, None] - lab) % L == 0)
    out = []
    for labelled in (True, False):
        print(f"[levels] ring of {L} labelled={labelled}", flush=True)
        ctx = F.Context(1, n_tau=6, nodes_per_panel=3)
        if labelled:
            ctx.set_momentum(0, *s.momentum)
        ctx.set_hamiltonian(0, s.h, s.eri, s.eps)
        out.append(ctx.eval_residual(0, s.mu, s.beta, t1, t2))
        ctx.close()
    for a, b in zip(*out):
        assert _close(a, b)


@pytest.mark.parametrize("L", [64, 66, 98])
def test_wide_wave_tiles_over_long_inner_ranges(F, L):
    """The same with one panel node: L ceil(L / 16)^2 >= 256 tiles of 16 x 16, so the 32 x 32
    wave tiles are taken; whole tiles over one batch of 64 inner indices, remainders of 2 in
    both, and three tiles and a remainder over a range that 16 x 16 tiles would split."""
    assert L * ((L + 15) // 16) ** 2 >= 256
    s = fi.hubbard_config(L=L, U=2.0, T=1.0)
    lab = np.arange(L)
    t1, t2 = fi.random_amplitudes(L, seed=L, scale=0.05)
    t1 = np.diag(np.diag(t1))
    t2 *= (lab[:, None, None, None] + lab[:, None, None] - lab[:, None] - lab) % L == 0
    out = []
    for labelled in (True, False):
        print(f"[levels] ring of {L}, one node, labelled={labelled}", flush=True)
        ctx = F.Context(1, n_tau=1, nodes_per_panel=1)
        if labelled:
            ctx.set_momentum(0, *s.momentum)
        ctx.set_hamiltonian(0, s.h, s.eri, s.eps)
        out.append(ctx.eval_residual(0, s.mu, s.beta, t1, t2))
        ctx.close()
    for a, b in zip(*out):
        assert _close(a, b)

"""The fused alpha and gamma kernels with chirp convolutions, and scales that go through a stage
together: a real signal against the same signal as a complex one (reality=False: the kernel that
takes two maps, other orders side by side), and both against the persistent executor, which runs
the separate passes one scale at a time.

Sizes: every transform size (128 .. 8192), 1 .. 4 orders side by side or in several passes, four
and eight samples per thread, the last band-limit of a size and the first of the next, scales
too large to go together (L = 1500, N = 8), blocked transforms (L = 512 and more), both full grids and the multiresolution one."""
import numpy as np
import pytest
import torch

from paper_1308_5706_amd import s2dw

pytestmark = pytest.mark.gpu

# two roundings of the same sums of FP64 (FP32) convolutions of at most 8192 points after the same
# Wigner sums, relative to the largest value
TOL = {"fp64": 1e-11, "mixed": 1e-5}


def real_signal(L, seed):
    """f_lm of a real signal: f_{l,-m} = (-1)^m conj f_lm."""
    g = np.random.default_rng(seed)
    f = np.zeros(L * L, complex)
    for el in range(L):
        c = (g.standard_normal(el + 1) + 1j * g.standard_normal(el + 1)) / (el + 1)
        c[0] = c[0].real
        m = np.arange(el + 1)
        f[el * el + el + m] = c
        f[el * el + el - m[1:]] = (1 - 2 * (m[1:] % 2)) * np.conj(c[1:])
    return torch.as_tensor(f, device="cuda")


def rel(a, b):
    return float((a - b).abs().max() / b.abs().max())


@pytest.mark.parametrize("L,N,J_min,grid", [
    (16, 3, 0, "mw"), (20, 3, 0, "mw"), (32, 8, 0, "mw"), (33, 2, 0, "mw"), (64, 7, 0, "mw"), (65, 5, 0, "mw"),
    (128, 1, 0, "mw"), (129, 8, 1, "mw"), (256, 6, 2, "mw"), (300, 6, 0, "mw"), (513, 3, 3, "mw"), (700, 8, 4, "mw"),
    (1024, 7, 5, "mw"), (1024, 2, 5, "mw"), (600, 5, 3, "mw"),
    (1100, 7, 7, "mw"), (1500, 8, 9, "mw"), (2047, 2, 9, "mw"), (31, 4, 0, "dh"), (150, 8, 2, "dh"), (512, 3, 4, "dh"),
    (90, 7, 0, "multires"), (300, 4, 2, "multires")])
def test_fused_equals_separate_passes(L, N, J_min, grid):
    print(f"L={L} N={N} J_min={J_min} {grid}", flush=True)
    f = real_signal(L, 7 * L + N)
    for prec, tol in TOL.items():
        kw = dict(precision=prec, grid=grid)
        W, Wp = s2dw.analysis(f, L, N, 2.0, J_min, **kw)
        Wc, Wpc = s2dw.analysis(f, L, N, 2.0, J_min, reality=False, **kw)
        assert rel(W, Wc.real) < tol and rel(Wp, Wpc) < tol
        b = s2dw.synthesis(W, Wp, L, N, 2.0, J_min, **kw)
        bc = s2dw.synthesis(W.to(Wc.dtype), Wp, L, N, 2.0, J_min, reality=False, **kw)
        assert rel(b, bc) < tol
        assert rel(b, f) < 100 * tol if prec == "fp64" else rel(b, f) < 10 * tol
        del W, Wc


def test_batches_beside_and_beyond_the_shared_workspace():
    # one and three maps of L = 40 go together, and the timed call's separate passes agree bitwise
    L, N = 40, 6
    f = torch.stack([real_signal(L, i) for i in range(3)])
    W, Wp = s2dw.analysis_batched(f, L, N, 2.0, 0)
    b = s2dw.synthesis_batched(W, Wp, L, N, 2.0, 0)
    s2dw.profile(True)
    try:
        W2, _ = s2dw.analysis(f[1], L, N, 2.0, 0)
        b2 = s2dw.synthesis(W2, Wp[1], L, N, 2.0, 0)
    finally:
        s2dw.profile(False)
    assert torch.equal(W[1], W2) and torch.equal(b[1], b2)


@pytest.mark.parametrize("L,N,J_min", [(18, 4, 0), (33, 8, 0), (64, 3, 0), (65, 7, 1), (130, 1, 2), (257, 8, 4), (500, 5, 6)])
def test_complex_signals_equal_two_real_ones_in_separate_passes(L, N, J_min):
    print(f"L={L} N={N} J_min={J_min}", flush=True)
    a, b = real_signal(L, 1), real_signal(L, 2)
    ab = torch.stack([a, b])
    for prec, tol in TOL.items():
        W, Wp = s2dw.analysis(a + 1j * b, L, N, 2.0, J_min, precision=prec, reality=False)
        (Wr, Wpr), = s2dw.analysis_persistent([(L, N, 2.0, J_min, ab)], precision=prec)
        assert rel(W.real, Wr[0]) < tol and rel(W.imag, Wr[1]) < tol
        assert rel(Wp, Wpr[0] + 1j * Wpr[1]) < tol
        c = s2dw.synthesis(W, Wp, L, N, 2.0, J_min, precision=prec, reality=False)
        cr, = s2dw.synthesis_persistent([(L, N, 2.0, J_min, Wr, Wpr)], precision=prec)
        assert rel(c, cr[0] + 1j * cr[1]) < tol
        W2 = s2dw.analysis(b, L, N, 2.0, J_min, precision=prec)[0]
        assert rel(W2, Wr[1]) < tol

"""Every Wigner tile shape (m' slots per wave) against the CPU reference, at band-limits and wavelet
parameters whose scale boundaries fall inside the kernels' blocks of eight l-steps.

The analysis sums do not depend on the shape (bitwise); the synthesis sums differ by the
grouping of the m'-sum only."""
import numpy as np
import pytest
import torch

import oracle
from paper_1308_5706_amd import s2dw
from paper_1308_5706_amd.inputs import random_flm

pytestmark = pytest.mark.gpu

TOL = 1e-11


def rel(x, ref):
    return np.max(np.abs(x - ref)) / np.max(np.abs(ref))


# N = 1 .. 16 covers every number of carried orders; (L, lam) put band-limits at 1, 2, 4, 7, 9, 11, ..
@pytest.mark.parametrize("L,N,lam", [(9, 1, 2.0), (23, 2, 3.0), (65, 3, 2.0), (70, 4, 1.5), (66, 5, 3.0),
                                     (37, 8, 2.5), (40, 10, 2.0), (33, 12, 3.0), (35, 14, 2.0), (24, 16, 2.0)])
def test_every_tile_shape_matches_the_oracle(L, N, lam):
    print(f"L={L} N={N} lam={lam}", flush=True)
    f = random_flm(L, L)
    fd = torch.as_tensor(f, device="cuda")
    ref = oracle.analysis(f, L, N, lam, 0)
    s0, chunk, fuse = s2dw.get_tuning(L, N, lam, 0)
    W0, Wp = s2dw.analysis(fd, L, N, lam, 0)
    seen = 0
    try:
        for slots in (1, 2, 4):
            try:
                s2dw.set_tuning(L, N, lam, 0, slots=slots, chunk=chunk, fuse=fuse)
            except s2dw.S2DWError:
                continue
            seen += 1
            W, _ = s2dw.analysis(fd, L, N, lam, 0)
            back = s2dw.synthesis(W0, Wp, L, N, lam, 0)
            assert torch.equal(W, W0)
            assert rel(W.cpu().numpy(), ref) < TOL
            assert rel(back.cpu().numpy(), f) < 1e-12
            Wm, Wpm = s2dw.analysis(fd, L, N, lam, 0, precision="mixed")
            backm = s2dw.synthesis(Wm, Wpm, L, N, lam, 0, precision="mixed")
            assert rel(backm.cpu().numpy(), f) < 1e-5
    finally:
        s2dw.set_tuning(L, N, lam, 0, slots=s0, chunk=chunk, fuse=fuse)
    assert seen >= 1


def test_batch_takes_another_shape_with_the_same_results():
    # one map of L = 130 runs one slot per wave, forty run two: bitwise the same
    L, N, B = 130, 5, 40
    f = torch.stack([torch.as_tensor(random_flm(L, i), device="cuda") for i in range(B)])
    W, _ = s2dw.analysis_batched(f, L, N, 2.0, 1)
    for i in (0, 17, B - 1):
        assert torch.equal(s2dw.analysis(f[i], L, N, 2.0, 1)[0], W[i])

"""The analysis that allocates nothing at the largest sizes whose arrays fit its scratch (one scale
and order: the least other arrays beside the rows of f_lm; many scales: the most rows), against the allocating call, bitwise,
and the first sizes beyond."""
import ctypes

import pytest
import torch

from paper_1308_5706_amd import s2dw
from paper_1308_5706_amd.inputs import random_flm, random_flm_complex

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,reality,lam,J_min,fits", [
    (832, 1, True, 2.0, 10, True), (833, 1, True, 2.0, 10, False),
    (586, 1, False, 2.0, 10, True), (587, 1, False, 2.0, 10, False),
    (389, 2, False, 1.2, 10, True)])  # the most rows beyond L
def test_largest_sizes_of_the_scratch(L, N, reality, lam, J_min, fits):
    print(f"L={L} N={N} reality={reality} lam={lam} J_min={J_min}", flush=True)
    f = torch.as_tensor((random_flm if reality else random_flm_complex)(L, L), device="cuda")
    A = (L, N, lam, J_min)
    ref, ref_phi = s2dw.analysis(f, *A, reality=reality)
    W, phi = torch.full_like(ref, float("nan")), torch.full_like(ref_phi, float("nan"))
    p = s2dw.params(L, N, lam, J_min, "fp64", "mw", reality)
    rc = s2dw.lib().s2dw_analysis_noalloc(ctypes.byref(p), ctypes.c_void_p(f.data_ptr()), ctypes.c_void_p(W.data_ptr()),
                                          ctypes.c_void_p(phi.data_ptr()),
                                          ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert rc == (0 if fits else -4)
    if fits:
        assert torch.equal(W, ref) and torch.equal(phi, ref_phi)
    s2dw.release_caches()

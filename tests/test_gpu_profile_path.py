"""Timing the stages times the program that runs without it: the smallest maps, whose scales go
through the fused alpha and gamma kernels, are reported as those, at every size."""
import pytest
import torch

from paper_1308_5706_amd import s2dw
from paper_1308_5706_amd.inputs import random_flm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("L,N", [(40, 3), (48, 8), (63, 4), (64, 4), (100, 7)])
def test_timed_calls_take_the_fused_kernels(L, N, precision):
    print(f"timed stages L={L} N={N} {precision}", flush=True)
    A = (L, N, 2.0, 0)
    S = s2dw.num_scales(L, 2.0, 0)
    f = torch.as_tensor(random_flm(L, L), device="cuda")
    ref, ref_phi = s2dw.analysis(f, *A, precision=precision)
    back = s2dw.synthesis(ref, ref_phi, *A, precision=precision)
    try:
        s2dw.profile_stages(None)
        s2dw.profile(True)
        W, Wp = s2dw.analysis(f, *A, precision=precision)
        out = s2dw.synthesis(W, Wp, *A, precision=precision)
        every = s2dw.profile_read()
        s2dw.profile_stages(["alpha_gamma_fwd"])
        s2dw.profile(True)
        s2dw.analysis(f, *A, precision=precision)
        some = s2dw.profile_read()
    finally:
        s2dw.profile(False)
        s2dw.profile_stages(None)
    assert every["alpha_gamma_fwd"][1] == every["gamma_alpha_adj"][1] == S
    for stage in ("alpha_fwd", "gamma_fwd", "gamma_adj", "alpha_adj"):
        assert every[stage] == (0.0, 0), stage
    assert set(some) == {"alpha_gamma_fwd"} and some["alpha_gamma_fwd"][1] == S
    assert torch.equal(W, ref) and torch.equal(out, back)

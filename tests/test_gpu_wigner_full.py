"""The synthesis Wigner kernel's form for launches of more workgroups than CUs (four waves per SIMD): the
maps of such a batch bitwise equal to single calls, which take the ordinary form, at band-limits
and dilations whose scale boundaries fall inside the kernels' blocks of eight l-steps; and a single
map large enough to take it, with start values below the double range, by its round trip."""
import pytest
import torch

from paper_1308_5706_amd import s2dw
from paper_1308_5706_amd.inputs import random_flm

pytestmark = pytest.mark.gpu


# FP64 with one and two carried orders (N = 1 .. 4), mixed precision with seven and eight (N = 13 .. 16):
# ceil(L / 64) ceil(L / 8) workgroups per map
@pytest.mark.parametrize("L,N,lam,J_min,B,precision", [
    (64, 1, 2.0, 0, 64, "fp64"), (70, 2, 1.5, 0, 24, "fp64"), (66, 3, 3.0, 0, 24, "fp64"), (130, 4, 2.0, 1, 8, "fp64"),
    (50, 13, 1.5, 0, 40, "mixed"), (64, 14, 2.0, 1, 40, "mixed"), (41, 15, 3.0, 0, 48, "mixed"),
    (100, 16, 2.0, 2, 12, "mixed")])
def test_batches_equal_single_calls(L, N, lam, J_min, B, precision):
    print(f"L={L} N={N} lam={lam} B={B} {precision}", flush=True)
    tiles = -(-L // 64) * -(-L // 8)
    assert tiles <= 256 < tiles * B
    A = (L, N, lam, J_min)
    f = torch.stack([torch.as_tensor(random_flm(L, i), device="cuda") for i in range(B)])
    W, Wp = s2dw.analysis_batched(f, *A, precision=precision)
    back = s2dw.synthesis_batched(W, Wp, *A, precision=precision)
    for i in (0, B // 2, B - 1):
        assert torch.equal(back[i], s2dw.synthesis(W[i].clone(), Wp[i], *A, precision=precision)), i
    assert float((back - f).abs().max() / f.abs().max()) < (1e-12 if precision == "fp64" else 1e-5)


@pytest.mark.parametrize("N", [14, 16])
def test_one_large_map_in_mixed_precision(N):
    L, J_min = 1100, 10
    print(f"L={L} N={N}", flush=True)
    f = torch.as_tensor(random_flm(L, N), device="cuda")
    W, Wp = s2dw.analysis(f, L, N, 2.0, J_min, precision="mixed")
    back = s2dw.synthesis(W, Wp, L, N, 2.0, J_min, precision="mixed")
    assert float((back - f).abs().max() / f.abs().max()) < 1e-5
    del W
    s2dw.release_caches()
    torch.cuda.empty_cache()

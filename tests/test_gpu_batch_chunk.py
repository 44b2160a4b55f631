"""Batches around the number of maps whose scales go through each stage together (their beta-stage
arrays fit 512 MiB side by side): the chunk's workspace, and each map's result bitwise that of the
single call on both sides of the line."""
import pytest
import torch

from paper_1308_5706_amd import s2dw
from paper_1308_5706_amd.inputs import random_flm, random_flm_complex

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,N,J_min,grid", [(536, 1, 3, "mw"), (576, 1, 0, "mw"), (504, 1, 3, "mw"), (512, 8, 1, "mw"),
                                            (400, 3, 2, "dh"), (500, 2, 1, "multires")])
def test_default_chunk_fits_its_workspace(L, N, J_min, grid):
    print(f"L={L} N={N} J_min={J_min} {grid}", flush=True)
    s2dw.release_caches()
    assert s2dw.workspace_bytes(L, N, 2.0, J_min, count=64, grid=grid) <= 8 << 30
    chunk = s2dw.get_tuning(L, N, 2.0, J_min, grid=grid)[1]
    one = s2dw.workspace_bytes(L, N, 2.0, J_min, count=1, grid=grid)
    assert chunk == 64 or (chunk + 2) * one > 8 << 30  # and is not smaller than it need be
    s2dw.release_caches()


# 512 MiB hold 21 maps of L = 256, N = 8 (a complex signal is two maps), 13 on the Driscoll-Healy grid
# of L = 230 and 39 of L = 536, N = 1: a batch on either side of the line
@pytest.mark.parametrize("L,N,J_min,grid,reality,below,beyond", [
    (256, 8, 0, "mw", True, 20, 24), (230, 8, 0, "dh", True, 13, 18), (256, 8, 0, "mw", False, 10, 12),
    (536, 1, 3, "mw", True, 38, 41),
    # batches whose alpha and gamma sums go in two passes (analysis of three scales with five and
    # more orders; synthesis on grids of their own), a single call's in one launch or one kernel
    (100, 10, 5, "mw", True, 8, 50), (129, 6, 6, "multires", True, 8, 20), (65, 8, 5, "multires", False, 8, 20)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_maps_of_a_batch_equal_single_calls_across_the_line(L, N, J_min, grid, reality, below, beyond, precision):
    print(f"L={L} N={N} {grid} reality={reality} {precision}", flush=True)
    A = (L, N, 2.0, J_min)
    kw = dict(precision=precision, grid=grid, reality=reality)
    f = torch.stack([torch.as_tensor((random_flm if reality else random_flm_complex)(L, i), device="cuda")
                     for i in range(beyond)])
    for count in (below, beyond):
        W, Wp = s2dw.analysis_batched(f[:count], *A, **kw)
        back = s2dw.synthesis_batched(W, Wp, *A, **kw)
        for i in (0, count // 2, count - 1):
            W1, Wp1 = s2dw.analysis(f[i], *A, **kw)
            assert torch.equal(W[i], W1) and torch.equal(Wp[i], Wp1), (count, i)
            assert torch.equal(back[i], s2dw.synthesis(W1, Wp1, *A, **kw)), (count, i)
        del W, Wp, back
    s2dw.release_caches()
    torch.cuda.empty_cache()

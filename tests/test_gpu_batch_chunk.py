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

"""Reading a tuning and applying it: an identity, for the default tile shape (whose slots follow
direction, precision and size) and for one that was set, in either precision.  The sums of the
synthesis are rounded by groups of m', so that a shape shows in its bits."""
import pytest
import torch

from paper_1308_5706_amd import s2dw
from paper_1308_5706_amd.inputs import random_flm

pytestmark = pytest.mark.gpu

PRECISIONS = ("fp64", "mixed")


def state(f, A):
    """What every tuning query reports, and the syntheses of both precisions."""
    out = {}
    for prec in PRECISIONS:
        W, Wp = s2dw.analysis(f, *A, precision=prec)
        out[prec] = (s2dw.get_tuning(*A, precision=prec), s2dw.synthesis(W, Wp, *A, precision=prec))
    return out


def same(a, b):
    return all(a[p][0] == b[p][0] and torch.equal(a[p][1], b[p][1]) for p in PRECISIONS)


def apply(A, prec, t):
    s2dw.set_tuning(*A, slots=t[0], chunk=t[1], fuse=t[2], precision=prec)


# carried orders 1, 2, 3 and 4, with one slot in FP64 and another number in mixed precision; then
# sizes with the same number in both
@pytest.mark.parametrize("L,N", [(100, 1), (90, 4), (70, 5), (100, 8), (60, 10), (600, 4)])
def test_applying_the_tuning_that_was_read_changes_nothing(L, N):
    print(f"tuning L={L} N={N}", flush=True)
    A = (L, N, 2.0, 2)
    f = torch.as_tensor(random_flm(L, L + N), device="cuda")
    s2dw.release_caches()
    default = state(f, A)
    for prec in PRECISIONS:
        apply(A, prec, default[prec][0])
        assert same(state(f, A), default), prec
    for prec in PRECISIONS:
        for slots in (1, 2, 4):
            try:
                apply(A, prec, (slots,) + default[prec][0][1:])
            except s2dw.S2DWError:
                continue
            assert s2dw.get_tuning(*A, precision=prec)[0] == slots
            now = state(f, A)
            for q in PRECISIONS:
                apply(A, q, now[q][0])
                assert same(state(f, A), now), (prec, slots, q)
            apply(A, prec, default[prec][0])  # and back
            assert same(state(f, A), default), (prec, slots)
    s2dw.autotune(*A, count=2)
    tuned = state(f, A)
    for prec in PRECISIONS:
        apply(A, prec, tuned[prec][0])
        assert same(state(f, A), tuned), prec
    s2dw.release_caches()

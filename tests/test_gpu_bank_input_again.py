"""The filter bank's input gradient on the matrix cores where its sums are not finite (NaN, infinities, sums past the
scaled range): those pixels are taken again by FMAs, with the FMA tiles' values, at a bounded cost."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

from oracle import oracle  # noqa: E402
from paper_1605_06399_amd import binding as B  # noqa: E402
from test_gpu_bank_input_mfma import cu, forced, index, problem  # noqa: E402

if gpu_available():
    import torch
    from paper_1605_06399_amd import torch_api as T


def same_kind(fma, got):
    assert np.array_equal(np.isnan(fma), np.isnan(got)) and np.array_equal(np.isinf(fma), np.isinf(got))
    inf = np.isinf(fma)
    assert np.array_equal(fma[inf], got[inf])


@pytest.mark.parametrize("r", [3, 4])
@pytest.mark.parametrize("H,W", [(1, 8), (5, 130), (40, 127), (33, 260), (300, 140)])
def test_values(r, H, W):
    gy, w = problem(2, 5, H, W, r)
    for s in (1e30, 1e36):   # whole sums past the range; finite, and some of them infinite in float32
        big = (s * gy).astype(np.float32)
        with np.errstate(over="ignore"):
            ref = oracle.bank_bwd_input(big, w).reshape(2, H, W)
            mag = oracle.bank_bwd_input(np.abs(big), np.abs(w)).reshape(2, H, W)
        got = forced(index(), cu(big), cu(w))
        ok = mag < 1e38   # no partial sum overflows
        assert np.all(np.abs(got[ok] - ref[ok]) <= 1e-5 * mag[ok])
        scaled = forced(index(), cu(big), cu(w), scale=torch.full((1,), 0.5, device="cuda"))
        assert np.array_equal(scaled[ok], np.float32(0.5) * got[ok])
    for v in (np.nan, np.inf):
        full = np.full_like(gy, v)
        same_kind(forced(2, cu(full), cu(w)), forced(index(), cu(full), cu(w)))
        few = gy.copy()
        few.reshape(2, 5, -1)[0, 3, [0, H * W // 2, H * W - 1]] = v
        same_kind(forced(2, cu(few), cu(w)), forced(index(), cu(few), cu(w)))
    # an infinite tap: positions outside the image do not count, as in the plain kernel (the tiles multiply it with the
    # zeros they stage there); the outermost pixels are the border kernel's
    taps = w.copy()
    taps[1, 0, 2 * r] = np.inf
    same_kind(*(forced(v, cu(gy), cu(taps))[:, 1:-1, 1:-1] for v in (0, index())))


def time_us(v, gy, w):
    B.check(B.icl_force_variant(B.ICL_OP_BANK_BWD_INPUT, v))
    try:
        T.bank_bwd_input(gy, w)
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(4):
            T.bank_bwd_input(gy, w)
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) * 250.0
    finally:
        B.icl_force_variant(B.ICL_OP_BANK_BWD_INPUT, -1)


@pytest.mark.parametrize("value", [float("nan"), float("inf"), 1e30, 1e-40])
def test_cost_does_not_depend_on_the_values_without_bound(value):
    """A step whose gradients overflowed: every pixel is taken again.  The same FMAs as the tiles' without their staging:
    within 12 times their time (taken pixel by pixel they were 140 times)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    w = 0.1 * torch.randn(16, 9, 9, generator=g, device="cuda")
    gy = value * torch.randn(4, 16, 1024, 1024, generator=g, device="cuda")
    assert time_us(index(), gy, w) <= 12.0 * time_us(2, gy, w)

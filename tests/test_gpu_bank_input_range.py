"""The filter bank's input gradient on the matrix cores over float32's range: small gradients under large taps and the
reverse, subnormal values, filters whose magnitudes lie 2^180 apart, against the FP64 oracle."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

from oracle import oracle  # noqa: E402
from paper_1605_06399_amd import synth  # noqa: E402
from test_gpu_bank_input_mfma import cu, forced, index  # noqa: E402

if gpu_available():
    import torch

F, H, W = 16, 24, 150


def check(gy, w):
    """Float32 sums of F (2r+1)^2 terms: 1e-5 of the sum of magnitudes as for every variant of this operation, and one
    rounding of a subnormal result.  The image's outermost pixels are another kernel's (the folds), which sums by FMAs
    and rounds each of a subnormal sum's terms: they are not looked at here."""
    ref, mag = (f(gy, w).reshape(H, W) for f in (oracle.bank_bwd_input, lambda a, b: oracle.bank_bwd_input(np.abs(a), np.abs(b))))
    got = forced(index(), cu(gy), cu(w))[0].astype(np.float64)
    got, ref, mag = (a[1:-1, 1:-1] for a in (got, ref, mag))
    assert np.all(np.abs(got - ref) <= 1e-5 * mag + 2.0 ** -149), np.max(np.abs(got - ref) / mag)


def problem(r, sg, sw):
    k = 2 * r + 1
    gy = sg * synth.normal(synth.seed(77, r), F * H * W).reshape(1, F, H, W).astype(np.float64)
    w = sw * synth.normal(synth.seed(78, r), F * k * k).reshape(F, k, k).astype(np.float64)
    return gy, w


@pytest.mark.parametrize("r", [3, 4])
@pytest.mark.parametrize("sg,sw", [(1e-35, 1e9), (1e-36, 1e10), (1e-37, 1e12), (1e25, 1e-37), (1e-42, 1e30), (1e30, 1e-42),
                                   (1e-43, 1.0), (1.0, 1e-43), (1e-20, 1e-21)])
def test_small_and_large_operands(r, sg, sw):
    gy, w = problem(r, sg, sw)
    check(gy.astype(np.float32), w.astype(np.float32))


@pytest.mark.parametrize("r", [3, 4])
def test_callers_factor(r):
    """The same products, the factor rounded into them once: factors around the smallest that takes the scaling in."""
    gy, w = (a.astype(np.float32) for a in problem(r, 1.0, 1.0))
    one = forced(index(), cu(gy), cu(w))
    for f in (0.3, -7e20, 2.0 ** -78, 3e-24, -1e-30, 0.0):
        got = forced(index(), cu(gy), cu(w), scale=torch.full((1,), f, device="cuda"))
        assert np.array_equal(got, np.float32(f) * one), f


@pytest.mark.parametrize("r", [3, 4])
def test_filters_of_different_magnitudes(r):
    gy, w = problem(r, 1.0, 1.0)
    e = 2.0 ** np.linspace(-90, 90, F).round()
    check((gy * e[None, :, None, None]).astype(np.float32), (w / e[:, None, None]).astype(np.float32))

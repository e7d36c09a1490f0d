"""The filter bank's input gradient on the matrix cores: strips of 128 columns and their tails, few and many rows (one
and several row blocks), filter counts up to the 16 of a product, infinities, NaN and values at the ends of float32's
range, against the FP64 oracle; the default's choice."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

from oracle import oracle  # noqa: E402
from paper_1605_06399_amd import binding as B, synth  # noqa: E402

if gpu_available():
    import torch
    from paper_1605_06399_amd import torch_api as T

NAME = "mfma_bf16x3_fold"


def index():
    names = [B.icl_variant_name(B.ICL_OP_BANK_BWD_INPUT, v) for v in range(B.icl_variant_count(B.ICL_OP_BANK_BWD_INPUT))]
    return names.index(NAME)


def forced(v, gy, w, scale=None):
    B.check(B.icl_force_variant(B.ICL_OP_BANK_BWD_INPUT, v))
    try:
        return T.bank_bwd_input(gy, w, scale=scale).cpu().numpy()[:, 0]
    finally:
        B.icl_force_variant(B.ICL_OP_BANK_BWD_INPUT, -1)


def cu(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def problem(N, F, H, W, r, s=1.0):
    k = 2 * r + 1
    gy = (s * synth.normal(synth.seed(75, r), N * F * H * W)).reshape(N, F, H, W).astype(np.float32)
    w = synth.normal(synth.seed(76, r), F * k * k).reshape(F, k, k).astype(np.float32)
    return gy, w


# float32 sums of F (2r+1)^2 terms: 1e-5 of the sum of magnitudes, as for the other variants of this operation
@pytest.mark.parametrize("N,F,H,W", [(1, 16, 1, 8), (1, 1, 9, 9), (2, 3, 5, 127), (1, 8, 17, 128), (1, 16, 40, 129),
                                     (2, 15, 33, 131), (1, 16, 300, 260), (3, 9, 70, 384)])
@pytest.mark.parametrize("r", [3, 4])
def test_matches_the_oracle(N, F, H, W, r):
    gy, w = problem(N, F, H, W, r)
    ref = oracle.bank_bwd_input(gy, w)
    mag = oracle.bank_bwd_input(np.abs(gy), np.abs(w))
    got = forced(index(), cu(gy), cu(w))
    assert np.max(np.abs(got - ref.reshape(got.shape)) / np.where(mag == 0, 1, mag).reshape(got.shape)) <= 1e-5
    half = forced(index(), cu(gy), cu(w), scale=torch.full((1,), 0.5, device="cuda"))
    assert np.array_equal(half, np.float32(0.5) * got)


@pytest.mark.parametrize("r", [3, 4])
def test_special_values(r):
    gy, w = problem(1, 12, 40, 200, r)
    gy[0, 3, 20, 70], gy[0, 5, 9, 130], gy[0, 7, 30, 12], gy[0, 1, 31, 150] = np.inf, -np.inf, np.nan, 3.4e38
    fma, got = forced(2, cu(gy), cu(w)), forced(index(), cu(gy), cu(w))
    assert np.array_equal(np.isnan(fma), np.isnan(got)) and np.array_equal(np.isfinite(fma), np.isfinite(got))
    inf = np.isinf(fma)
    assert inf.any() and np.array_equal(fma[inf], got[inf])
    for s in (1e-37, 1e-33, 1e30):
        gy, w = problem(1, 16, 20, 140, r, s)
        ref = oracle.bank_bwd_input(gy, w).reshape(20, 140)
        mag = oracle.bank_bwd_input(np.abs(gy), np.abs(w)).reshape(20, 140)
        assert np.max(np.abs(forced(index(), cu(gy), cu(w))[0] - ref) / mag) <= 1e-5, s


def test_default_choice():
    for (n, f, h, w, r, name) in [(32, 16, 1024, 1024, 4, NAME), (32, 11, 1024, 1024, 4, "pers_p4x4_fold"),
                                  (1, 16, 512, 512, 4, "pers_p4x4_fold"), (32, 16, 1024, 1024, 2, "pers_p4x4_fold"),
                                  (60, 16, 1024, 150, 4, "pers_p4x4_fold"), (32, 17, 1024, 1024, 4, "tile64_p4x4_fold")]:
        st, v = B.icl_selected_variant_problem(B.ICL_OP_BANK_BWD_INPUT, B.ICL_F32, r, w, h, n=n, f=f)
        B.check(st)
        assert B.icl_variant_name(B.ICL_OP_BANK_BWD_INPUT, v) == name, (n, f, h, w, r)
    assert B.icl_variant_arith(B.ICL_OP_BANK_BWD_INPUT, index()) == "bf16x3_mfma"

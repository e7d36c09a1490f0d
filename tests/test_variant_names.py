"""What an unforced, untuned call runs is reported under the name of the kernel that runs (CPU: selection needs no
device)."""
import pytest

from paper_1605_06399_amd import binding as B


def selected(op, dtype, r, w, h, **kw):
    st, v = B.icl_selected_variant_problem(op, dtype, r, w, h, **kw)
    assert st == B.ICL_OK
    return B.icl_variant_name(op, v)


@pytest.mark.parametrize("dtype,r,w,h,name", [
    (B.ICL_F32, 7, 4096, 4096, "pers_p8x4"), (B.ICL_F32, 5, 4096, 2048, "pers_p8x4"), (B.ICL_F32, 5, 4095, 2048, "pers_p4x2"),
    (B.ICL_F32, 4, 4096, 4096, "pers_p4x2"), (B.ICL_F32, 0, 1, 1, "pers_p4x2"), (B.ICL_F16, 7, 4096, 4096, "pers_p4x2"),
    (B.ICL_BF16, 3, 640, 480, "pers_p4x2"), (B.ICL_F16, 2, 4096, 4096, "lds_p4x2_o1"), (B.ICL_BF16, 0, 5, 5, "lds_p4x2_o1")])
def test_2d_correlation(dtype, r, w, h, name):
    assert selected(B.ICL_OP_CONV2D, dtype, r, w, h) == name
    assert B.icl_selected_variant(B.ICL_OP_CONV2D, dtype, r, w, h) == (B.ICL_OK, 1)   # the untuned mark
    assert B.icl_variant_name(B.ICL_OP_CONV2D, 1) == "lds_p4x4_o0"

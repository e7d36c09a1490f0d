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


@pytest.mark.parametrize("r,w,name", [(0, 512, "strip_p4_t16"), (1, 512, "mfma_i8"), (4, 16, "mfma_i8"), (4, 15, "strip_p4_t16"),
                                      (5, 512, "mfma_i8"), (7, 16, "mfma_i8"), (7, 15, "plain")])
def test_unsigned_char_correlation(r, w, name):
    assert selected(B.ICL_OP_CONV2D_U8, B.ICL_U8, r, w, 512) == name
    v = B.icl_selected_variant(B.ICL_OP_CONV2D_U8, B.ICL_U8, r, w, 512)[1]
    assert B.icl_variant_name(B.ICL_OP_CONV2D_U8, v) == name


@pytest.mark.parametrize("r,w,name", [(1, 256, "strips_any_t8"), (1, 255, "row4"), (1, 1, "row4"), (2, 512, "plain")])
def test_nms(r, w, name):
    assert selected(B.ICL_OP_NMS, B.ICL_F32, r, w, 512) == name


@pytest.mark.parametrize("op,dtype,r,w,h,kw,entry,name", [
    # the tuned entry's own kernel takes the call: it runs
    (B.ICL_OP_CONV2D_U8, B.ICL_U8, 5, 512, 512, {}, "plain", "plain"),
    (B.ICL_OP_BANK_BWD_INPUT, B.ICL_F32, 3, 512, 512, {"n": 2, "f": 8}, "mfma_bf16x3_fold", "mfma_bf16x3_fold"),
    # it does not: the default runs, not another kernel under the entry's name
    (B.ICL_OP_CONV2D_U8, B.ICL_U8, 2, 15, 512, {}, "mfma_i8", "strip_p4_t16"),
    (B.ICL_OP_BANK_BWD_INPUT, B.ICL_F32, 2, 512, 512, {"n": 2, "f": 8}, "mfma_bf16x3_fold", "pers_p4x4_fold"),
    (B.ICL_OP_BANK_BWD_INPUT, B.ICL_F32, 4, 512, 512, {"n": 2, "f": 17}, "mfma_bf16x3_fold", "tile64_p4x4_fold"),
    (B.ICL_OP_BANK_BWD_INPUT, B.ICL_F32, 4, 7, 512, {"n": 2, "f": 8}, "mfma_bf16x3_fold", "pers_p4x4_fold")])
def test_tuned_entries(tmp_path, op, dtype, r, w, h, kw, entry, name):
    names = {B.ICL_OP_CONV2D_U8: "conv2d_u8", B.ICL_OP_BANK_BWD_INPUT: "bank_bwd_input"}
    size = (w * h * kw.get("n", 1)).bit_length() - 1
    p = tmp_path / "cache.json"
    for device in ("unknown|0", "gfx950|256"):
        p.write_text('{"version": 1, "entries": [\n  {"key": "%s|%s|%d|%d|%d|f%d|m0", "variant": "%s", "us": 1.0}\n]}\n'
                     % (device, names[op], dtype, r, size, kw.get("f", 1), entry))
        assert B.icl_tune_load(str(p)) == B.ICL_OK
    try:
        assert selected(op, dtype, r, w, h, **kw) == name
    finally:
        B.icl_tune_clear()

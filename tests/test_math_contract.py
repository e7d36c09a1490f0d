"""The header's arithmetic contract names what runs: every arithmetic that selection may pick in the default mode stands
in the paragraph of ICL_MATH_F32 (CPU; the variant tables need no device)."""
import os
import re

from paper_1605_06399_amd import binding as B

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "icl.h")


def test_every_default_arithmetic_is_named():
    with open(HEADER) as f:
        text = f.read()
    f32 = re.search(r"ICL_MATH_F32 \(the default\):(.*?)ICL_MATH_F16_SPLIT:", text, re.S).group(1)
    split = re.search(r"ICL_MATH_F16_SPLIT: (.*?)The mode is process-wide", text, re.S).group(1)
    assert '"mfma_f16x3"' in split and '"fp16x3_mfma"' not in f32
    seen = set()
    for op in range(B.ICL_OP_CONV3D_SEP + 1):
        if op == B.ICL_OP_CONV2D_U8:   # integers
            continue
        for v in range(B.icl_variant_count(op)):
            seen.add(B.icl_variant_arith(op, v))
    assert {"fp32_valu", "fp32_mfma", "fp16x3_mfma"} <= seen
    for arith in seen - {"fp16x3_mfma"}:
        assert f'"{arith}"' in f32, f"{arith} runs by default and the contract does not name it"

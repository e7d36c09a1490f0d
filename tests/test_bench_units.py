"""bench.py measures every phase of the training step against the unit its kernel runs on (CPU)."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402
from paper_1605_06399_amd import binding as B  # noqa: E402


def test_unit_peaks():
    assert bench.unit_peak_tflops("fp32_valu") == 78.6 and bench.unit_peak_tflops("fp32_mfma") == 157.3
    # six products of bfloat16 parts for one of float32: no phase can exceed it, as one did against the FMA units' peak
    assert abs(bench.unit_peak_tflops("bf16x3_mfma") - 2500.0 / 6.0) < 1e-9
    for op in (B.ICL_OP_BANK_FWD, B.ICL_OP_BANK_FWD_SSE, B.ICL_OP_BANK_BWD_INPUT, B.ICL_OP_BANK_BWD_FILTER):
        for v in range(B.icl_variant_count(op)):
            assert bench.unit_peak_tflops(B.icl_variant_arith(op, v)) > 0

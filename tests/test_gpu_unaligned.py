"""GPU parity at the edges of the vector staging: rows that start at any element, image widths around
4 pixels and around a tile, sources and destinations that are views into a larger buffer (nothing outside
the destination's rows may change), both boundaries, every variant, against the FP64 oracle."""
import numpy as np
import pytest

from conftest import gpu_available
from helpers import assert_close, empty_padded, padded_view, storage

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

from oracle import oracle  # noqa: E402
from paper_1605_06399_amd import binding as B, synth  # noqa: E402

if gpu_available():
    import torch
    from paper_1605_06399_amd import torch_api as T

WIDTHS = [1, 2, 3, 4, 5, 7, 63, 65, 67, 130]


def dev_taps(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize("border", ["clamp", "constant"])
@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("op", ["sep", "2d"])
def test_any_width_and_offset(op, dt, border):
    r, H, c = 3, 37, 0.5
    n = 2 * r + 1
    h, v = (synth.normal_taps_normalised(61, n, stream=q) for q in (0, 1))
    w = synth.normal_taps_normalised(61, n * n, stream=2).reshape(n, n)
    code = B.ICL_OP_CONV_SEP if op == "sep" else B.ICL_OP_CONV2D
    for k, W in enumerate(WIDTHS):
        xd, x64 = storage(synth.image_uniform(62 + k, H, W) + 0.25, dt)
        src = padded_view(xd, pad_elems=1 + k % 3, offset_elems=1 + k % 5)
        if op == "sep":
            ref = oracle.conv_sep(x64, h, v, border=border, constant=c)
            S = oracle.normwise_scale_sep(x64, h, v, border=border, constant=c)
        else:
            ref = oracle.conv2d(x64, w, border=border, constant=c)
            S = oracle.normwise_scale_conv2d(x64, w, border=border, constant=c)
        ws = torch.empty(H * W + 1, dtype=torch.float32, device="cuda")
        for i in range(B.icl_variant_count(code)):
            out = empty_padded(H, W, src.dtype, pad_elems=2, offset_elems=3 - k % 3)
            B.check(B.icl_force_variant(code, i))
            try:
                if op == "sep":
                    T.conv_sep(src, dev_taps(h), dev_taps(v), out=out, workspace=ws, border=border, constant=c)
                else:
                    T.conv2d(src, dev_taps(w), out=out, border=border, constant=c)
            finally:
                B.icl_force_variant(code, -1)
            torch.cuda.synchronize()
            assert_close(out, ref, S, dt, f"{op} variant {i} {dt} {border} W={W}")
            whole = out._base
            inside = torch.zeros_like(whole, dtype=torch.bool)
            inside[out.storage_offset():out.storage_offset() + H * (W + 2)].view(H, W + 2)[:, :W] = True
            assert torch.isnan(whole[~inside]).all(), f"{op} variant {i} W={W}: wrote outside its rows"

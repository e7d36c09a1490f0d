"""The matrix-core walk of the unsigned char correlation, byte for byte against the oracle where it can go
wrong: widths around 16 bytes, a chunk and a 256-column strip, one row to several segments, rows at any
byte, both boundaries, taps whose high part is 128 (32640 and up), and the unforced calls of radius 5..7."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

from oracle import oracle  # noqa: E402
from paper_1605_06399_amd import binding as B, synth  # noqa: E402

if gpu_available():
    import torch
    from paper_1605_06399_amd import torch_api as T

SHAPES = [(1, 16), (2, 17), (9, 31), (40, 255), (17, 257), (33, 271), (70, 530), (3, 1025)]


@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 6, 7])
def test_bytes_equal_the_oracle(r):
    n = 2 * r + 1
    fixed = synth.u8_taps(80 + r, r, synth.U8_SHIFT)
    high = fixed.copy()
    high[0, 0], high[r, r], high[n - 1, n - 1] = 32767, 32640, -32768
    assert r > 4 or B.icl_variant_name(B.ICL_OP_CONV2D_U8, B.icl_selected_variant(
        B.ICL_OP_CONV2D_U8, B.ICL_U8, r, 512, 512)[1]) == "mfma_i8"
    for k, (H, W) in enumerate(SHAPES):
        X = synth.u8_image(81 + k, H, W)
        pad, off = 1 + k % 4, k % 5
        buf = torch.zeros((H + 1) * (W + pad) + off, dtype=torch.uint8, device="cuda")
        x = buf[off:off + H * (W + pad)].view(H, W + pad)[:, :W]
        x.copy_(torch.from_numpy(X))
        whole = torch.full((H, W + pad + 1), 0xA5, dtype=torch.uint8, device="cuda")
        for taps, shift in ((fixed, synth.U8_SHIFT), (high, 16), (high, 0)):
            td = torch.from_numpy(taps).cuda()
            for border, c in (("clamp", 0), ("constant", 0), ("constant", 201)):
                T.conv2d_u8(x, td, shift, out=whole[:, :W], border=border, constant=c)
                got = whole.cpu().numpy()
                ref = oracle.conv2d_u8(X, taps, shift, border=border, constant=c)
                assert np.array_equal(got[:, :W], ref), f"r{r} {H}x{W} shift {shift} {border} {c}"
                assert np.all(got[:, W:] == 0xA5), f"r{r} {H}x{W}: wrote outside the rows"

"""The unsigned char walk inside wide images: strips whose reads and writes all lie in the rows (two of them and more,
destination rows on four bytes), heights of one row, less than a ring of rows and several segments, every radius,
against the oracle; nothing outside the rows may change."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

from oracle import oracle  # noqa: E402
from paper_1605_06399_amd import synth  # noqa: E402

if gpu_available():
    import torch
    from paper_1605_06399_amd import torch_api as T


@pytest.mark.parametrize("H,W,pad", [(1, 776, 0), (9, 1024, 8), (40, 776, 4), (133, 1029, 3)])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 6, 7])
def test_inside_strips(r, H, W, pad):
    taps = synth.u8_taps(85, r, synth.U8_SHIFT)
    td = torch.from_numpy(taps).cuda()
    X = synth.u8_image(86 + r, H, W)
    x = torch.from_numpy(X).cuda()
    assert (W + pad) % 4 == 0
    for border, c in (("clamp", 0), ("constant", 201)):
        whole = torch.full((H, W + pad), 0xA5, dtype=torch.uint8, device="cuda")
        T.conv2d_u8(x, td, synth.U8_SHIFT, out=whole[:, :W], border=border, constant=c)
        got = whole.cpu().numpy()
        ref = oracle.conv2d_u8(X, taps, synth.U8_SHIFT, border=border, constant=c)
        assert np.array_equal(got[:, :W], ref), f"{border}"
        assert np.all(got[:, W:] == 0xA5), "wrote outside the rows"

"""GPU parity of the strips of the corner and NMS kernels where they can go wrong: rows that start at any byte,
widths around a strip's 256 (mask) or 240 (corners) columns and around the four pixels of a lane, heights around
a strip's rows, outputs that are views (nothing outside them may change), NaN and infinite responses.
Masks and the responses of the corner strips are compared exactly."""
import numpy as np
import pytest

from conftest import gpu_available
from helpers import padded_view, storage

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

from oracle import oracle  # noqa: E402
from paper_1605_06399_amd import binding as B, synth  # noqa: E402

if gpu_available():
    import torch
    from paper_1605_06399_amd import torch_api as T

TAU = np.float32(1e-3)


def mask_view(H, W, pad, off):
    buf = torch.full((H * (W + pad) + off + 8,), 7, dtype=torch.uint8, device="cuda")
    view = buf[off:off + H * (W + pad)].view(H, W + pad)[:, :W]
    return buf, view


def untouched(buf, H, W, pad, off):
    keep = torch.ones_like(buf, dtype=torch.bool)
    keep[off:off + H * (W + pad)].view(H, W + pad)[:, :W] = False
    return bool((buf[keep] == 7).all())


@pytest.mark.parametrize("pad,off,mpad,moff", [(0, 0, 0, 0), (1, 1, 3, 1), (3, 2, 1, 2)])
@pytest.mark.parametrize("W", [253, 255, 256, 257, 258, 259, 260, 511, 513, 770])
def test_nms_strips_any_rows(W, pad, off, mpad, moff):
    for H in (1, 2, 9, 10, 11, 33):
        u = synth.uniform01(synth.seed(61, W), H * W).reshape(H, W)
        q = ((np.floor(u * 6) - 1) * 1e-3).astype(np.float32)    # many ties
        q[u < 0.01] = np.inf
        q[(u > 0.01) & (u < 0.02)] = -np.inf
        q[(u > 0.02) & (u < 0.03)] = np.nan
        R = padded_view(torch.from_numpy(q).cuda(), pad, off)
        buf, out = mask_view(H, W, mpad, moff)
        T.nms(R, float(TAU), 1, out=out)
        assert np.array_equal(out.cpu().numpy(), oracle.nms(q, float(TAU))), f"{H}x{W}"
        assert untouched(buf, H, W, mpad, moff), f"{H}x{W}: bytes outside the mask changed"


@pytest.mark.parametrize("rg", [0, 1, 2, 3])
@pytest.mark.parametrize("W,pad,off", [(247, 0, 0), (248, 1, 1), (488, 3, 2), (489, 0, 3), (731, 2, 1)])
def test_corner_strip_heights_agree(rg, W, pad, off):
    g = torch.from_numpy(synth.gaussian_taps(rg, 1.0)).cuda()
    for H in (1, 4, 5, 13, 22, 37):
        xd, _ = storage(synth.image_uniform(62 + rg, H, W), "f32")
        x = padded_view(xd, pad, off)
        ref = None
        for variant in range(1, B.icl_variant_count(B.ICL_OP_CORNERS)):
            name = B.icl_variant_name(B.ICL_OP_CORNERS, variant)
            R = torch.empty((H, W), dtype=torch.float32, device="cuda")
            buf, out = mask_view(H, W, pad, off)
            B.check(B.icl_force_variant(B.ICL_OP_CORNERS, variant))
            try:
                T.corners(x, g, 0.04, float(TAU), resp=R, out=out)
            finally:
                B.icl_force_variant(B.ICL_OP_CORNERS, -1)
            assert untouched(buf, H, W, pad, off), f"{name} {H}x{W}: bytes outside the mask changed"
            assert np.array_equal(out.cpu().numpy(), oracle.nms(R.cpu().numpy(), float(TAU))), f"{name} {H}x{W}"
            if ref is None:
                ref = R
            assert torch.equal(R.view(torch.int32), ref.view(torch.int32)), f"{name} {H}x{W}: response bits"


@pytest.mark.parametrize("rg", [0, 1, 2, 3])
@pytest.mark.parametrize("W,pad,off", [(3, 0, 0), (251, 1, 1), (256, 0, 0), (260, 4, 0), (499, 0, 3), (503, 1, 0), (752, 0, 0)])
def test_harris_strip_heights_agree(rg, W, pad, off):
    """Every column has one rounding whatever the strip's height: the tile kernel's for rows off 16 bytes and, of
    aligned rows, for the left 4 columns and those right of the last whole strip."""
    g = synth.gaussian_taps(rg, 1.0)
    taps = torch.from_numpy(g).cuda()
    names = [B.icl_variant_name(B.ICL_OP_HARRIS, v) for v in range(B.icl_variant_count(B.ICL_OP_HARRIS))]
    aligned = W >= 256 and (W + pad) % 4 == 0 and off % 4 == 0 and W % 4 == 0
    xr = 4 + (W - 8) // 248 * 248
    for H in (1, 3, 4, 5, 11, 22, 37):
        xd, x64 = storage(synth.image_uniform(66 + rg, H, W), "f32")
        x = padded_view(xd, pad, off)
        out = {}
        for v, name in enumerate(names):
            if not (name == "fused_t16" or name.startswith("strips") or (aligned and name.startswith("stream"))):
                continue
            R = torch.empty((H, W), dtype=torch.float32, device="cuda")
            B.check(B.icl_force_variant(B.ICL_OP_HARRIS, v))
            try:
                T.harris(x, taps, out=R)
            finally:
                B.icl_force_variant(B.ICL_OP_HARRIS, -1)
            out[name] = R.view(torch.int32)
        bound = oracle.harris_f32_bound(x64, g, 0.04)
        err = np.abs(out["strips_t8"].view(torch.float32).cpu().numpy() - oracle.harris(x64, g, 0.04))
        assert (err <= bound).all(), f"{H}x{W}"
        for name, R in out.items():
            if name != "fused_t16":
                assert torch.equal(R, out["strips_t8"]), f"{name} {H}x{W}"
        tile = out["fused_t16"]
        if aligned:
            assert torch.equal(out["strips_t8"][:, :4], tile[:, :4]) and torch.equal(out["strips_t8"][:, xr:], tile[:, xr:])
        else:
            assert torch.equal(out["strips_t8"], tile), f"{H}x{W}"

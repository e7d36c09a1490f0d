"""The filter gradient's walk over 64 x 16 tiles (its choice for problems of few tiles): one tile to several
per work-group, ragged columns and rows, odd widths, every radius, 1 and 16 filters, against the oracle with
the bank's float32 normwise tolerance (the scale is the adjoint evaluated on absolute values)."""
import numpy as np
import pytest

from conftest import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]

from oracle import oracle  # noqa: E402
from paper_1605_06399_amd import binding as B, synth  # noqa: E402

if gpu_available():
    import torch
    from paper_1605_06399_amd import torch_api as T


@pytest.mark.parametrize("r", [1, 2, 3, 4])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (1, 2, 3, 2), (2, 16, 16, 64), (3, 5, 17, 65), (2, 3, 130, 33),
                                   (1, 7, 300, 203)])
def test_filter_gradient_of_few_tiles(shape, r):
    n, f, h, w = shape
    k = 2 * r + 1
    x = synth.normal(synth.seed(90, r), n * h * w).reshape(n, 1, h, w)
    gy = synth.normal(synth.seed(91, r), n * f * h * w).reshape(n, f, h, w)
    names = B.variant_names(B.ICL_OP_BANK_BWD_FILTER)
    st, v = B.icl_selected_variant_problem(B.ICL_OP_BANK_BWD_FILTER, B.ICL_F32, r, w, h, n=n, f=f)
    assert st == B.ICL_OK and names[v] == "mfma_walk_t64x16"
    gyd, xd = torch.from_numpy(gy).cuda(), torch.from_numpy(x).cuda()
    gw = T.bank_bwd_filter(gyd, xd, r)
    assert torch.equal(gw, T.bank_bwd_filter(gyd, xd, r))   # fixed order: the same bits again
    ref = oracle.bank_bwd_filter(gy, x, r).reshape(f, k, k)
    scale = oracle.bank_bwd_filter(np.abs(gy), np.abs(x), r).reshape(f, k, k)
    assert np.all(np.abs(gw.cpu().numpy().astype(np.float64) - ref) <= 1e-5 * scale)

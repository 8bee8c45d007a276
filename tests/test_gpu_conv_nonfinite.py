"""Weight gradients of layers whose input holds infinities and NaN at the box's
edges: a weight's sum is affected exactly where the definition says, also on
extents that leave bricks ragged, where positions beyond the box take part in
the matrix products with a zero gradient."""
import ctypes as C

import numpy as np
import pytest

from test_gpu_surrogate import _gpu, bft  # noqa: F401  (_gpu: the module fixture)

pytestmark = pytest.mark.gpu

# (n, d, h, w): ragged in x, in y, in both, in z alone, for the 16-, 8- and 4-wide
# bricks, one without ragged bricks, and one with enough positions for the forms of
# two output (and input) blocks per workgroup
SHAPES = [(1, 4, 4, 17), (1, 4, 5, 16), (2, 5, 7, 9), (1, 6, 8, 8), (1, 9, 3, 5), (1, 3, 6, 3), (1, 4, 4, 16),
          (1, 20, 22, 30), (1, 40, 41, 45)]


@pytest.mark.parametrize("pmask", [0, 1, 6])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("ci,co", [(16, 16), (32, 32), (16, 32)])
def test_weight_gradient_takes_nonfinite_inputs_where_they_belong(shape, ci, co, pmask):
    import torch
    from oracle import conv_ref as R
    from paper_1904_03618_amd import surrogate as S
    rng = np.random.default_rng([*shape, ci, co, pmask])
    layer = S.Conv("t", ci, co, 3, False, rng)
    n, d, h, w = shape
    a = rng.standard_normal(shape + (ci,)).astype(np.float32)
    a[0, d // 2, h // 2, w - 1, 1] = np.inf
    a[0, d // 2, h - 1, w // 2, 3] = np.nan
    a[n - 1, d - 1, h - 1, w - 1, 6] = -np.inf
    xt, x64 = bft(a)
    dyt, dy64 = bft(rng.standard_normal(shape + (co,)))
    ws = torch.full((int(S.lib().sg_conv3d_bwd_weight_ws(C.byref(S.view(dyt)), ci, 3)) // 4 + 1,), np.nan, device="cuda")
    layer.bwd_weight(S.view(xt), S.view(dyt), ws, pmask=pmask)
    got, gb = layer.gw.cpu().numpy(), layer.gb.cpu().numpy()
    with np.errstate(invalid="ignore"):
        dW, db = R.conv3d_bwd_weight(x64, dy64, k=3, pmask=pmask)
    ok = np.isfinite(dW)
    assert 0 < ok.sum() < dW.size
    assert np.array_equal(np.isfinite(got), ok)
    # FP32 sums of at most P products (2e-5 of the largest, as for finite inputs)
    assert np.abs(got[ok] - dW[ok]).max() <= 2e-5 * np.abs(dW[ok]).max()
    assert np.abs(gb - db).max() <= 2e-5 * np.abs(db).max()

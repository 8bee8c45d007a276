"""The 3x3x3 convolution and its weight gradient on extents that are no
multiples of their bricks (16, 8 and 4 wide, 256 or 512 positions), for every
kernel form the channel counts and sizes select, against the FP64 reference.
Inputs are BF16 values, so what remains is FP32 accumulation: at most K = 27 ci
(forward) or P (weight gradient) products summed in blocks, within 2e-5 of the
largest result."""
import ctypes as C

import numpy as np
import pytest

from test_gpu_surrogate import _gpu, bft, close  # noqa: F401  (_gpu: the module fixture)

pytestmark = pytest.mark.gpu

# extents (n, d, h, w): below a brick, one over it, each of the three brick
# widths padding least, a 1-wide axis
SHAPES = [(1, 1, 1, 1), (2, 3, 5, 2), (1, 5, 7, 9), (1, 8, 9, 8), (1, 4, 5, 17), (2, 9, 4, 16), (1, 4, 16, 24),
          (1, 2, 8, 4)]
# channels: one, two, three and four 8-channel groups per chunk, several chunks,
# one and two blocks of outputs
CHANNELS = [(8, 16), (16, 32), (24, 16), (56, 32), (64, 48), (96, 32)]


def _layer(ci, co, rng, k=3):
    import torch
    from paper_1904_03618_amd import surrogate as S
    layer = S.Conv("t", ci, co, k, False, rng)
    layer.b.copy_(torch.tensor(rng.standard_normal(co).astype(np.float32)))
    layer.prep()
    W64 = layer.w.to(torch.bfloat16).float().cpu().numpy().astype(np.float64)
    return layer, W64, layer.b.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("ci,co", CHANNELS)
def test_ragged_convolution_and_weight_gradient(shape, ci, co):
    import torch
    from oracle import conv_ref as R
    from paper_1904_03618_amd import surrogate as S
    for pmask in (3, 4):
        rng = np.random.default_rng([*shape, ci, co, pmask])
        layer, W64, b64 = _layer(ci, co, rng)
        xt, x64 = bft(rng.standard_normal(shape + (ci,)))
        y32 = torch.full(shape + (co,), np.nan, device="cuda")
        layer.fwd(S.view(xt), None, S.view(y32), pmask=pmask)
        ok, err = close(y32.cpu().numpy(), R.conv3d(x64, W64, b64, k=3, pmask=pmask))
        assert ok, ("fwd", pmask, err)
        dyt, dy64 = bft(rng.standard_normal(shape + (co,)))
        ws = torch.full((int(S.lib().sg_conv3d_bwd_weight_ws(C.byref(S.view(dyt)), ci, 3)) // 4 + 1,), np.nan,
                        device="cuda")
        layer.bwd_weight(S.view(xt), S.view(dyt), ws, pmask=pmask)
        dW, db = R.conv3d_bwd_weight(x64, dy64, k=3, pmask=pmask)
        ok, err = close(layer.gw.cpu().numpy(), dW)
        ok2, err2 = close(layer.gb.cpu().numpy(), db)
        assert ok and ok2, ("weight gradient", pmask, err, err2)


# large enough (above 131072 positions x 16 outputs) for the forms without
# weights in LDS; widths on which the 16-, 8- and 4-wide bricks pad least
@pytest.mark.parametrize("shape", [(1, 34, 64, 64), (1, 36, 70, 56), (1, 33, 64, 68)])
@pytest.mark.parametrize("ci,co", [(8, 16), (16, 16), (40, 32), (32, 16), (32, 32)])
def test_large_ragged_convolution_at_sampled_positions(shape, ci, co):
    import torch
    from oracle import conv_ref as R
    from paper_1904_03618_amd import surrogate as S
    n, d, h, w = shape
    assert n * d * h * w // 256 * (co // 16) > 512
    rng = np.random.default_rng([*shape, ci, co])
    layer, W64, b64 = _layer(ci, co, rng)
    xt, x64 = bft(rng.standard_normal(shape + (ci,)))
    y32 = torch.full(shape + (co,), np.nan, device="cuda")
    layer.fwd(S.view(xt), None, S.view(y32), pmask=3)
    pts = np.stack([rng.integers(0, s_, 400) for s_ in shape], axis=1)
    pts = np.concatenate([pts, [(0, 0, 0, 0), (0, d - 1, h - 1, w - 1), (0, 0, h - 1, 0), (0, d - 1, 0, w - 1)]])
    assert bool(torch.isfinite(y32).all())
    got = y32.cpu().numpy()[pts[:, 0], pts[:, 1], pts[:, 2], pts[:, 3]]
    ok, err = close(got, R.conv3d_at(x64, W64, pts, b64, k=3, pmask=3))
    assert ok, err


# several bricks per position group (more than 768 or 512 workgroups' worth)
@pytest.mark.parametrize("shape", [(2, 33, 64, 64), (1, 40, 72, 88)])
@pytest.mark.parametrize("ci,co", [(16, 16), (16, 32), (32, 32)])
def test_weight_gradient_of_large_ragged_layers(shape, ci, co):
    import torch
    from oracle import conv_ref as R
    from paper_1904_03618_amd import surrogate as S
    rng = np.random.default_rng([*shape, ci, co])
    layer, _, _ = _layer(ci, co, rng)
    xt, x64 = bft(rng.standard_normal(shape + (ci,)))
    dyt, dy64 = bft(rng.standard_normal(shape + (co,)))
    ws = torch.full((int(S.lib().sg_conv3d_bwd_weight_ws(C.byref(S.view(dyt)), ci, 3)) // 4 + 1,), np.nan,
                    device="cuda")
    layer.bwd_weight(S.view(xt), S.view(dyt), ws, pmask=3)
    dW, db = R.conv3d_bwd_weight(x64, dy64, k=3, pmask=3)
    ok, err = close(layer.gw.cpu().numpy(), dW)
    ok2, err2 = close(layer.gb.cpu().numpy(), db)
    assert ok and ok2, (err, err2)


@pytest.mark.parametrize("shape,ci,co", [((1, 1, 1, 3), 8, 4), ((2, 5, 7, 9), 24, 16), ((4, 20, 20, 20), 16, 4)])
def test_pointwise_weight_gradient(shape, ci, co):
    """1x1x1 layers: 256 consecutive positions per brick, a last partial one,
    several groups."""
    import torch
    from oracle import conv_ref as R
    from paper_1904_03618_amd import surrogate as S
    rng = np.random.default_rng([*shape, ci, co])
    layer, _, _ = _layer(ci, co, rng, k=1)
    xt, x64 = bft(rng.standard_normal(shape + (ci,)))
    dyt, dy64 = bft(rng.standard_normal(shape + (layer.co8,)))
    ws = torch.full((int(S.lib().sg_conv3d_bwd_weight_ws(C.byref(S.view(dyt, 0, co)), ci, 1)) // 4 + 1,), np.nan,
                    device="cuda")
    layer.bwd_weight(S.view(xt), S.view(dyt, 0, co), ws, pmask=3)
    dW, db = R.conv3d_bwd_weight(x64, dy64[..., :co], k=1, pmask=3)
    ok, err = close(layer.gw.cpu().numpy(), dW)
    ok2, err2 = close(layer.gb.cpu().numpy(), db)
    assert ok and ok2, (err, err2)


@pytest.mark.parametrize("shape", [(1, 4, 4, 16), (1, 3, 5, 9)])
def test_outputs_that_start_off_a_vector_boundary(shape):
    """Output tensors aligned to one value only: the same results as aligned
    ones, bit for bit, and nothing written beside them."""
    import torch
    from paper_1904_03618_amd import surrogate as S
    rng = np.random.default_rng(shape)
    layer, _, _ = _layer(16, 16, rng)
    xt, _ = bft(rng.standard_normal(shape + (16,)))
    n = int(np.prod(shape)) * 16
    y, y32 = (torch.zeros(shape + (16,), dtype=d, device="cuda") for d in (torch.bfloat16, torch.float32))
    layer.fwd(S.view(xt), S.view(y), S.view(y32), pmask=3)
    bufs = [torch.full((n + 16,), 7.0, dtype=t.dtype, device="cuda") for t in (y, y32)]
    oy, o32 = (b[1:1 + n].view(shape + (16,)) for b in bufs)
    layer.fwd(S.view(xt), S.view(oy), S.view(o32), pmask=3)
    assert torch.equal(oy, y) and torch.equal(o32, y32)
    for b in bufs:
        assert float(b[0]) == 7.0 and bool((b[1 + n:] == 7.0).all())

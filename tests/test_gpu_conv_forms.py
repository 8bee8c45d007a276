"""The forms of the convolution that its other tests do not reach: whole-brick
layers whose weights stay outside LDS, the 8-channel chunk, and inputs beyond the
32-bit offsets of the streaming form; and the loss over more positions than its
lanes take at once.  Against the FP64 reference at sampled positions (BF16 inputs,
FP32 sums of at most 27 ci products: within 2e-5 of the largest result)."""
import ctypes as C

import numpy as np
import pytest

from test_gpu_surrogate import _gpu, bft, close  # noqa: F401  (_gpu: the module fixture)

pytestmark = pytest.mark.gpu


def _layer(ci, co, rng, k=3):
    import torch
    from paper_1904_03618_amd import surrogate as S
    layer = S.Conv("t", ci, co, k, False, rng)
    layer.b.copy_(torch.tensor(rng.standard_normal(co).astype(np.float32)))
    layer.prep()
    W64 = layer.w.to(torch.bfloat16).float().cpu().numpy().astype(np.float64)
    return layer, W64, layer.b.cpu().numpy().astype(np.float64)


# (shape, ci, co): every extent a multiple of 16 x 4 x 4
#   8 -> 16: one 8-channel chunk, two planes per wave, a single brick and many
#   32 -> 16 and 64 -> 48 above 512 workgroups of one output block: no weights in
#     LDS, one block per workgroup (48 is no multiple of 32)
#   32 -> 32 and 96 -> 64 above that limit with d % 8 == 4: two blocks per workgroup
#   40 -> 16 with d % 8 == 4 above it: a last chunk of 8 channels
WHOLE = [((1, 8, 8, 16), 8, 16), ((2, 24, 20, 48), 8, 16), ((1, 40, 64, 64), 32, 16), ((1, 20, 64, 64), 64, 48),
         ((1, 36, 64, 48), 32, 32), ((1, 36, 32, 48), 96, 64), ((1, 36, 64, 64), 40, 16)]


@pytest.mark.parametrize("pmask", [3, 4])
@pytest.mark.parametrize("shape,ci,co", WHOLE)
def test_whole_brick_layers(shape, ci, co, pmask):
    import torch
    from oracle import conv_ref as R
    from paper_1904_03618_amd import surrogate as S
    n, d, h, w = shape
    assert w % 16 == 0 and h % 4 == 0 and d % 4 == 0
    if ci != 8:
        assert n * d * h * w // 256 * (co // 16) > 512
        assert co % 32 or d % 8 == 4
    rng = np.random.default_rng([*shape, ci, co])
    layer, W64, b64 = _layer(ci, co, rng)
    xt, x64 = bft(rng.standard_normal(shape + (ci,)))
    y, y32 = (torch.full(shape + (co,), np.nan, dtype=t, device="cuda") for t in (torch.bfloat16, torch.float32))
    layer.fwd(S.view(xt), S.view(y), S.view(y32), pmask=pmask)
    assert bool(torch.isfinite(y32).all()) and torch.equal(y, y32.to(torch.bfloat16))
    pts = np.stack([rng.integers(0, s_, 300) for s_ in shape], axis=1)
    pts = np.concatenate([pts, [(0, 0, 0, 0), (n - 1, d - 1, h - 1, w - 1), (0, 0, h - 1, 0), (0, d - 1, 0, w - 1)]])
    got = y32.cpu().numpy()[pts[:, 0], pts[:, 1], pts[:, 2], pts[:, 3]]
    ok, err = close(got, R.conv3d_at(x64, W64, pts, b64, k=3, pmask=pmask))
    assert ok, err


# both sides of the rule that sends a small layer's weights through LDS (more than
# 48 input channels with one output block per workgroup, more than 16 with two)
@pytest.mark.parametrize("shape", [(1, 4, 4, 16), (2, 12, 8, 32)])
@pytest.mark.parametrize("ci,co", [(8, 16), (48, 16), (56, 16), (64, 48), (16, 32), (32, 32), (40, 64)])
def test_small_whole_brick_layers(shape, ci, co):
    import torch
    from oracle import conv_ref as R
    from paper_1904_03618_amd import surrogate as S
    rng = np.random.default_rng([*shape, ci, co])
    layer, W64, b64 = _layer(ci, co, rng)
    xt, x64 = bft(rng.standard_normal(shape + (ci,)))
    for pmask in (3, 4):
        y32 = torch.full(shape + (co,), np.nan, device="cuda")
        layer.fwd(S.view(xt), None, S.view(y32), pmask=pmask)
        ok, err = close(y32.cpu().numpy(), R.conv3d(x64, W64, b64, k=3, pmask=pmask))
        assert ok, (pmask, err)


@pytest.mark.parametrize("co", [16, 32])
def test_inputs_of_two_gigabytes(co):
    """2^31 bytes of input on ragged extents: past the 32-bit byte offsets of the
    streaming form.  The definition is evaluated at sampled positions from the
    input values gathered there."""
    import torch
    from paper_1904_03618_amd import surrogate as S
    rng = np.random.default_rng(co)
    ci, shape = 8, (1, 513, 512, 515)
    n, d, h, w = shape
    assert d * h * w * ci * 2 >= 2 ** 31
    layer, W64, b64 = _layer(ci, co, rng)
    g = torch.Generator(device="cuda").manual_seed(co)
    x = torch.empty(shape + (ci,), dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    y = torch.empty(shape + (co,), dtype=torch.bfloat16, device="cuda")
    layer.fwd(S.view(x), S.view(y), pmask=1)               # periodic in x, zero beyond y and z
    pts = np.stack([rng.integers(0, s_, 200) for s_ in (d, h, w)], axis=1)
    pts = np.concatenate([pts, [(0, 0, 0), (d - 1, h - 1, w - 1), (d - 1, 0, 0), (256, h - 1, 0)]])
    taps = np.array([(z, yy, xx) for z in (-1, 0, 1) for yy in (-1, 0, 1) for xx in (-1, 0, 1)])
    q = pts[:, None, :] + taps
    q[..., 2] %= w
    inside = ((q >= 0) & (q < (d, h, w))).all(axis=2)
    i = torch.tensor(np.where(inside[..., None], q, 0), device="cuda")
    v = x[0, i[..., 0], i[..., 1], i[..., 2]].double().cpu().numpy() * inside[..., None]
    want = v.reshape(len(pts), -1) @ W64.T + b64
    p = torch.tensor(pts, device="cuda")
    got = y[0, p[:, 0], p[:, 1], p[:, 2]].double().cpu().numpy()
    # BF16 results: half a unit in the last of 8 bits, besides the sums' 2e-5
    assert np.abs(got - want).max() <= (2.0 ** -8 + 2e-5) * np.abs(want).max()


@pytest.mark.parametrize("ctot,coff", [(4, 0), (8, 4)])
def test_mse_over_more_positions_than_lanes(ctot, coff):
    """345 600 positions on 262 144 lanes: a second, partial trip."""
    import torch
    from oracle import conv_ref as R
    from paper_1904_03618_amd import surrogate as S
    rng = np.random.default_rng(ctot)
    shape = (2, 40, 60, 72)
    out, tgt, grad = (torch.tensor(rng.standard_normal(shape + (ctot,)).astype(np.float32), device="cuda")
                      for _ in range(3))
    loss = torch.zeros(257, dtype=torch.float64, device="cuda")
    v = lambda t: C.byref(S.view(t, coff, 4))
    assert S.lib().sg_mse(v(out), v(tgt), v(grad), C.c_void_p(loss.data_ptr()), S._stream()) == 0
    f64 = lambda t: t[..., coff:coff + 4].double().cpu().numpy()
    l64, g64 = R.mse(f64(out), f64(tgt))
    assert abs(loss[0].item() - l64) < 1e-6 * l64 and close(f64(grad), g64, 1e-6)[0]


# ragged layers of 32 outputs per workgroup on both sides of 1024 waves of one block
@pytest.mark.parametrize("shape,ci,co", [((1, 7, 33, 67), 24, 64), ((1, 9, 35, 53), 24, 64), ((2, 17, 19, 23), 16, 128)])
def test_ragged_layers_around_a_wave_per_simd(shape, ci, co):
    import torch
    from oracle import conv_ref as R
    from paper_1904_03618_amd import surrogate as S
    n, d, h, w = shape
    assert (n * d * h * w // 64 * (co // 16) >= 1024) == (shape != (1, 7, 33, 67))
    rng = np.random.default_rng([*shape, ci, co])
    layer, W64, b64 = _layer(ci, co, rng)
    xt, x64 = bft(rng.standard_normal(shape + (ci,)))
    y32 = torch.full(shape + (co,), np.nan, device="cuda")
    layer.fwd(S.view(xt), None, S.view(y32), pmask=3)
    ok, err = close(y32.cpu().numpy(), R.conv3d(x64, W64, b64, k=3, pmask=3))
    assert ok, err

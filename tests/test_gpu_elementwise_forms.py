"""The element-wise layers of the surrogate in each form their channels and
alignment select (8, 4 and 1 channels per thread, slices of wider arrays,
unaligned bases), against the FP64 reference; casts and copies bit for bit."""
import ctypes as C

import numpy as np
import pytest

from test_gpu_surrogate import _gpu, close  # noqa: F401  (_gpu: the module fixture)

pytestmark = pytest.mark.gpu

# channels, channels of the array, offset of the slice, elements the base is shifted by
FORMS = [(16, 16, 0, 0), (8, 24, 8, 0), (12, 20, 4, 0), (4, 8, 4, 0), (3, 5, 1, 0), (8, 8, 0, 1), (4, 8, 0, 3)]


def array(rng, shape, ctot, shift, dtype):
    """A CUDA array (shape + (ctot,)) whose base lies `shift` elements past an aligned one."""
    import torch
    n = int(np.prod(shape)) * ctot
    flat = torch.zeros(n + shift, dtype=dtype, device="cuda")
    t = flat[shift:].view(*shape, ctot)
    t.copy_(torch.tensor(rng.standard_normal(shape + (ctot,)).astype(np.float32)))
    return t


@pytest.mark.parametrize("c,ctot,coff,shift", FORMS)
def test_relu_backward_cast(c, ctot, coff, shift):
    import torch
    from paper_1904_03618_amd import surrogate as S
    rng = np.random.default_rng(c + ctot)
    shape = (2, 3, 5, 7)
    g = array(rng, shape, ctot, shift, torch.float32)
    y = array(rng, shape, ctot, shift, torch.bfloat16)
    for mask in (y, None):
        out = torch.full(shape + (ctot,), 7.0, dtype=torch.bfloat16, device="cuda")
        assert S.lib().sg_relu_bwd_cast(C.byref(S.view(g, coff, c)), C.byref(S.view(mask, coff, c)) if mask is not None
                                        else None, C.byref(S.view(out, coff, c)), S._stream()) == 0
        sl = slice(coff, coff + c)
        want = g[..., sl] if mask is None else torch.where(y[..., sl].float() > 0, g[..., sl], torch.zeros_like(g[..., sl]))
        assert torch.equal(out[..., sl], want.to(torch.bfloat16))
        rest = torch.ones(ctot, dtype=torch.bool)
        rest[sl] = False
        assert bool((out[..., rest] == 7.0).all())


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("c,ctot,coff,shift", FORMS)
def test_pool_and_upsampling_adjoints(c, ctot, coff, shift, accumulate):
    import torch
    from oracle import conv_ref as R
    from paper_1904_03618_amd import surrogate as S
    rng = np.random.default_rng(3 * c + ctot)
    fine, coarse = (2, 4, 6, 10), (2, 2, 3, 5)
    sl = slice(coff, coff + c)
    f64 = lambda t: t[..., sl].double().cpu().numpy()
    dy, dx = array(rng, coarse, ctot, shift, torch.float32), array(rng, fine, ctot, shift, torch.float32)
    want = R.pool2_bwd(f64(dy)) + (f64(dx) if accumulate else 0.0)
    assert S.lib().sg_pool2_bwd(C.byref(S.view(dy, coff, c)), C.byref(S.view(dx, coff, c)), accumulate, S._stream()) == 0
    assert close(f64(dx), want, 1e-6)[0]
    dy, dx = array(rng, fine, ctot, shift, torch.float32), array(rng, coarse, ctot, shift, torch.float32)
    want = R.up2_bwd(f64(dy)) + (f64(dx) if accumulate else 0.0)
    assert S.lib().sg_up2_bwd(C.byref(S.view(dy, coff, c)), C.byref(S.view(dx, coff, c)), accumulate, S._stream()) == 0
    assert close(f64(dx), want, 1e-6)[0]


@pytest.mark.parametrize("c,ctot,coff,shift", [(4, 4, 0, 0), (4, 8, 4, 0), (4, 4, 0, 1), (3, 5, 1, 0)])
@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (2, 20, 40, 44)])
def test_mse(shape, c, ctot, coff, shift):
    """One position, and more than the 256 x 1024 lanes take at once (with
    several values per lane)."""
    import torch
    from oracle import conv_ref as R
    from paper_1904_03618_amd import surrogate as S
    rng = np.random.default_rng(c + shape[1])
    out, tgt, grad = (array(rng, shape, ctot, shift, torch.float32) for _ in range(3))
    loss = torch.zeros(257, dtype=torch.float64, device="cuda")
    v = lambda t: C.byref(S.view(t, coff, c))
    assert S.lib().sg_mse(v(out), v(tgt), v(grad), C.c_void_p(loss.data_ptr()), S._stream()) == 0
    f64 = lambda t: t[..., coff:coff + c].double().cpu().numpy()
    l64, g64 = R.mse(f64(out), f64(tgt))
    assert abs(loss[0].item() - l64) < 1e-6 * l64 and close(f64(grad), g64, 1e-6)[0]


def test_adam_on_flat_parameters_equals_layer_by_layer():
    """The network's one launch over its flat arrays against a launch per tensor
    (bit for bit: the step is element-wise), also after a layer's tensor has been
    replaced by the caller."""
    import torch
    from paper_1904_03618_amd import surrogate as S
    a, b = (S.UNet((1, 8, 8, 8), seed=3) for _ in range(2))
    for n in (a, b):
        g = torch.Generator(device="cuda").manual_seed(1)
        for l in n.layers:
            l.gw.copy_(torch.randn(l.gw.shape, device="cuda", generator=g))
            l.gb.copy_(torch.randn(l.gb.shape, device="cuda", generator=g))
    first = b.layers[0]
    first.w, first.b = first.w.clone(), first.b.clone()          # b now steps tensor by tensor
    for _ in range(3):
        a.adam(1e-3)
        b.adam(1e-3)
    for la, lb in zip(a.layers, b.layers):
        for x, y in ((la.w, lb.w), (la.b, lb.b), (la.wb, lb.wb), (la.wt, lb.wt), (la.bias_pad, lb.bias_pad)):
            assert torch.equal(x, y), la.name

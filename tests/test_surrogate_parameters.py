"""Where the network's parameters live (host logic, no GPU: the library is
replaced by a stand-in that steps the memory it is handed).  Adam has to reach
every layer's arrays, and a layer's bias the array the kernels read, however the
network came by them: as built, copied, pickled, or with arrays of the caller's."""
import copy
import ctypes as C
import pickle

import numpy as np
import pytest
import torch

from paper_1904_03618_amd import surrogate as S

LR = 0.25


class Library:
    """w -= lr g, m = g, v = 2 g over the n floats at each address."""

    def __init__(self):
        self.launches = 0

    def sg_adam(self, w, g, m, v, n, lr, *rest):
        w, g, m, v = (np.ctypeslib.as_array((C.c_float * n).from_address(p.value)) for p in (w, g, m, v))
        w -= np.float32(lr) * g
        m[:], v[:] = g, 2 * g
        self.launches += 1
        return 0

    def sg_weight_prep(self, *args):
        return 0

    def sg_conv3d_bwd_weight_ws(self, *args):
        return 64


@pytest.fixture
def net(monkeypatch):
    zeros = torch.zeros
    monkeypatch.setattr(torch, "zeros", lambda *a, device=None, **kw: zeros(*a, **kw))
    fake = Library()
    monkeypatch.setattr(S, "lib", lambda: fake)
    monkeypatch.setattr(S, "_stream", lambda: None)
    n = S.UNet((1, 8, 8, 8), seed=3)
    n.fake = fake
    return n


def _own_storage(n):
    for t in n.layers[2].__dict__.values():
        if isinstance(t, torch.Tensor) and t.dtype == torch.float32:
            t.data = t.data.clone()
    return n


def _replaced(n):
    l = n.layers[4]
    l.w, l.b, l.gb = l.w.clone(), l.b.clone(), l.gb.clone()
    return n


def _before_flat(n):
    """As a network pickled before its arrays were flat: every layer its own."""
    del n.flat
    for l in n.layers:
        for k in ("w", "b", "gw", "gb", "mw", "mb", "vw", "vb", "bias_pad"):
            setattr(l, k, getattr(l, k).clone())
    return n


def _without_fake(n, f):
    fake = n.__dict__.pop("fake")
    out = f(n)
    out.fake = n.fake = fake
    return out


FORMS = {
    "as built": (lambda n: n, 1),
    "deep copy": (lambda n: _without_fake(n, copy.deepcopy), 1),
    "pickled": (lambda n: _without_fake(n, lambda m: pickle.loads(pickle.dumps(m))), 30),
    "tensor data replaced": (_own_storage, 30),
    "attributes replaced": (_replaced, 30),
    "without flat arrays": (_before_flat, 30),
    "a layer left out": (lambda n: (n.layers.pop(3), n)[1], 28),
}


@pytest.mark.parametrize("form", list(FORMS))
def test_adam_steps_every_layer(net, form):
    make, launches = FORMS[form]
    n = make(net)
    gen = torch.Generator().manual_seed(1)
    want = {}
    for l in n.layers:
        for t in (l.gw, l.gb):
            t.copy_(torch.randn(t.shape, generator=gen))
        want[l.name] = (l.w - LR * l.gw, l.b - LR * l.gb)
    n.fake.launches = 0
    n.adam(LR)
    for l in n.layers:
        w, b = want[l.name]
        assert torch.equal(l.w, w) and torch.equal(l.b, b), l.name
        assert torch.equal(l.mw, l.gw) and torch.equal(l.vb, 2 * l.gb), l.name
        assert torch.equal(l.bias_pad[:l.co], b) and not l.bias_pad[l.co:].any(), l.name
    assert n.fake.launches == launches


@pytest.mark.parametrize("form", list(FORMS))
def test_loaded_state_reaches_the_kernels(net, form):
    n = FORMS[form][0](net)
    rng = np.random.default_rng(5)
    sd = {l.name: (rng.standard_normal((l.co, l.K)).astype(np.float32), rng.standard_normal(l.co).astype(np.float32))
          for l in n.layers}
    n.load_state(sd)
    for l in n.layers:
        assert np.array_equal(l.w.numpy(), sd[l.name][0]), l.name
        assert np.array_equal(l.bias_pad[:l.co].numpy(), sd[l.name][1]), l.name

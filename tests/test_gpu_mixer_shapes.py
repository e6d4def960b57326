"""Mixer network at the edges of the fused pass: window columns that fill whole
blocks of 32, leave one column or several, partial blocks of hidden units,
partial blocks of sites, batches of one state and of more states than
workgroups, and the shapes beyond it (w > 64, h > 256).  Tolerances are those of
the network's other tests: FP32 products and sums of at most a few thousand
terms against FP64."""
import numpy as np
import pytest

from oracle import closed_form as cf
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,w,h,b", [(65, 0, 33, 2), (130, 16, 40, 5), (100, 15, 256, 1), (100, 64, 256, 2),
                                     (64, 5, 32, 300), (50, 65, 20, 2), (40, 5, 257, 2)])
def test_mixer_shapes(gpu, n, w, h, b):
    import torch

    from paper_2409_17033_amd.mixer import Mixer
    g = torch.Generator().manual_seed(n + w)
    u, en = 0.5 + torch.rand(n, generator=g), 2 * torch.rand(n, generator=g) - 1
    net = Mixer(u.to(gpu), en.to(gpu), window=w, hidden=h, seed=3)
    # every parameter away from zero (the biases start there)
    net.params.copy_((0.3 * torch.randn(net.count, generator=g)).bfloat16().view(torch.int16))
    x, t = torch.randn(b, n, generator=g), torch.randn(b, n, generator=g)
    p = net.params_float().double().cpu().numpy()
    args = (x.double().numpy(), u.double().numpy(), en.double().numpy(), w, h)
    yref, _, _ = omlp.forward(p, *args)
    assert cf.rel_frobenius(net.forward(x.to(gpu)).double().cpu().numpy(), yref) <= 1e-5
    loss, grad = net.loss_grad(x.to(gpu), t.to(gpu))
    lref, gref = omlp.loss_grad(p, args[0], t.double().numpy(), *args[1:])
    assert abs(loss - lref) <= 1e-5 * lref
    grad = grad.double().cpu().numpy()
    assert cf.rel_frobenius(grad, gref) <= 1e-4
    k = 4 * w + 3                                       # and each part of the gradient by itself
    for a, e in ((0, h * k), (h * k, h * k + h), (h * k + h, h * k + 2 * h), (h * k + 2 * h, h * k + 2 * h + 1)):
        assert cf.rel_frobenius(grad[a:e], gref[a:e]) <= 1e-3

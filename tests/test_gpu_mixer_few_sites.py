"""Mixer network with few sites and many states, on both sides of the rule that
sends such batches to the general products (forward: fewer than 16 sites and more
than 256 states; gradient: fewer than 4 and more than 1024): against the FP64
oracle with the tolerances of the network's other tests."""
import time

import numpy as np
import pytest

from oracle import closed_form as cf
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,w,h,b", [(15, 3, 20, 256), (15, 3, 20, 257), (16, 3, 20, 257), (3, 2, 40, 1024),
                                     (3, 2, 40, 1025), (4, 2, 40, 1025), (1, 0, 5, 2000)])
def test_few_sites(gpu, n, w, h, b):
    import torch

    from paper_2409_17033_amd.mixer import Mixer
    g = torch.Generator().manual_seed(n + b)
    u, en = 0.5 + torch.rand(n, generator=g), 2 * torch.rand(n, generator=g) - 1
    net = Mixer(u.to(gpu), en.to(gpu), window=w, hidden=h, seed=3)
    net.params.copy_((0.3 * torch.randn(net.count, generator=g)).bfloat16().view(torch.int16))
    x, t = torch.randn(b, n, generator=g), torch.randn(b, n, generator=g)
    p = net.params_float().double().cpu().numpy()
    args = (x.double().numpy(), u.double().numpy(), en.double().numpy(), w, h)
    yref, _, _ = omlp.forward(p, *args)
    assert cf.rel_frobenius(net.forward(x.to(gpu)).double().cpu().numpy(), yref) <= 1e-5
    loss, grad = net.loss_grad(x.to(gpu), t.to(gpu))
    lref, gref = omlp.loss_grad(p, args[0], t.double().numpy(), *args[1:])
    assert abs(loss - lref) <= 1e-5 * lref
    assert cf.rel_frobenius(grad.double().cpu().numpy(), gref) <= 1e-4


def test_many_states_of_one_site(gpu):
    """16384 states of one site have the rows of 256 states of 64 sites: the
    blocks of sites may not make them several times as long."""
    import torch

    from paper_2409_17033_amd.mixer import Mixer
    times = []
    for n, b in ((1, 16384), (64, 256)):
        g = torch.Generator(device=gpu).manual_seed(n)
        net = Mixer(torch.rand(n, device=gpu, generator=g), torch.rand(n, device=gpu, generator=g), window=8, hidden=64)
        x = torch.randn(b, n, device=gpu, generator=g)
        best = 1e9
        for _ in range(20):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            net.forward(x)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        times.append(1e6 * best)
    print(f"\none site {times[0]:.0f} us, 64 sites {times[1]:.0f} us")
    assert times[0] <= 2.5 * times[1]

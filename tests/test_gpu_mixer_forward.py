"""The forward pass of the mixer network does strictly less work than the loss
gradient, and one without a window less than one with: both have to show it.
Batches of several states per workgroup, so that the work per state counts."""
import time

import pytest

pytestmark = pytest.mark.gpu


def _best(f, reps=20):
    import torch
    best = 1e9
    for _ in range(reps):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        f()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t0)
    return best


@pytest.mark.parametrize("n,w,h,b", [(64, 8, 32, 4096), (64, 32, 100, 4096), (100, 2, 64, 2048)])
def test_forward_is_no_slower_than_the_gradient(gpu, n, w, h, b):
    import torch

    from paper_2409_17033_amd.mixer import Mixer
    g = torch.Generator(device=gpu).manual_seed(n)
    u, en = torch.rand(n, device=gpu, generator=g), torch.rand(n, device=gpu, generator=g)
    x, t = torch.randn(b, n, device=gpu, generator=g), torch.randn(b, n, device=gpu, generator=g)
    net, point = Mixer(u, en, window=w, hidden=h, seed=3), Mixer(u, en, window=0, hidden=h, seed=3)
    tf, tg, t0 = _best(lambda: net.forward(x)), _best(lambda: net.loss_grad(x, t)), _best(lambda: point.loss_grad(x, t))
    print(f"\nforward {1e6 * tf:.0f} us, gradient {1e6 * tg:.0f} us, without a window {1e6 * t0:.0f} us")
    assert tf <= 1.1 * tg and t0 <= 1.1 * tg

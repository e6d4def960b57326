"""An infinite or NaN input of the mixer network reaches the outputs of the sites
whose window holds it, and only those: not a site one past the window, not
through the padding of partial blocks of hidden units or sites.  Infinite hidden
sums have tanh = +-1, so outputs stay finite there, and gradients are finite but
for the columns that meet the infinity.  Which entries are finite, and their
values, are compared with the FP64 oracle (tolerances of the network's other
tests)."""
import numpy as np
import pytest

from oracle import closed_form as cf
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("where", ["x", "E"])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("n,w,h,site", [(100, 5, 40, 80), (100, 5, 40, 99), (100, 16, 64, 64), (70, 0, 3, 69), (128, 20, 32, 30),
                                          (40, 5, 40, 38), (20, 16, 33, 19), (100, 33, 32, 97), (50, 50, 20, 49)])
def test_reach_of_a_nonfinite_input(gpu, n, w, h, site, bad, where):
    import torch

    from paper_2409_17033_amd.mixer import Mixer
    g = torch.Generator().manual_seed(n + w)
    u, en = 0.5 + torch.rand(n, generator=g), 2 * torch.rand(n, generator=g) - 1
    x, t = torch.randn(3, n, generator=g), torch.randn(3, n, generator=g)
    if where == "x":
        x[1, site] = bad
    else:
        en[site] = bad
    net = Mixer(u.to(gpu), en.to(gpu), window=w, hidden=h, seed=3)
    net.params.copy_((0.3 * torch.randn(net.count, generator=g)).bfloat16().view(torch.int16))
    p = net.params_float().double().cpu().numpy()
    args = (x.double().numpy(), u.double().numpy(), en.double().numpy(), w, h)

    def same(got, ref):
        ok = np.isfinite(ref)
        assert (np.isfinite(got) == ok).all()
        if ok.any():
            assert cf.rel_frobenius(got[ok], ref[ok]) <= 1e-4

    with np.errstate(invalid="ignore"):
        yref, _, _ = omlp.forward(p, *args)
        lref, gref = omlp.loss_grad(p, args[0], t.double().numpy(), *args[1:])
    same(net.forward(x.to(gpu)).double().cpu().numpy(), yref)
    loss, grad = net.loss_grad(x.to(gpu), t.to(gpu))
    assert np.isfinite(loss) == np.isfinite(lref)
    same(grad.double().cpu().numpy(), gref)

"""One sweep step rounds each entry of Z = Y X + X Y once.  X_1 = I - H with a
projector H that pairs orbital i with i + n / 2 (entries +-1/2): a single step
with sigma = +1 then gives chi = -(A X + X A), whose entries are sums of four
halved entries of A.  The halves of a pair lie in different accumulation chains,
so that the chains are exact, and adding them in FP64 is exact too: the result is
the correctly rounded sum, bit for bit, for every tile size and number of waves
(the sizes below), on the diagonal tiles as off them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sweep", ["forward", "adjoint"])
@pytest.mark.parametrize("n,prec", [(128, "fp32"), (576, "fp32"), (832, "fp32"), (1000, "fp32"), (1280, "fp32"), (128, "split3_bf16"),
                                    (1024, "split3_bf16"), (128, "split_fp16"), (1024, "split_fp16")])
def test_step_rounds_once(gpu, n, prec, sweep):
    import torch

    import paper_2409_17033_amd as dm
    half = n // 2
    x = np.zeros((n, n))
    i = np.arange(half)
    x[i, i] = x[i + half, i + half] = 0.5
    x[i, i + half] = x[i + half, i] = -0.5
    rng = np.random.default_rng(n)
    # up to 20 significant bits (exact in every split), sizes over 2^12
    a = np.ldexp(rng.integers(-(1 << 20), 1 << 20, (n, n)).astype(np.float64), -20 - rng.integers(0, 12, (n, n)))
    a = np.trunc(np.ldexp(a, 24)) * 2.0 ** -24
    a = np.triu(a) + np.triu(a, 1).T
    h = (np.eye(n) - x).astype(np.float32)
    chi, d, _, info = dm.susceptibility(torch.from_numpy(h).to(gpu), torch.from_numpy(a.astype(np.float32)).to(gpu), half,
                                        precision=prec, sweep=sweep, bounds="given", emin=0.0, emax=1.0, min_iter=1,
                                        project=False, spin=1.0)
    assert info["m"] == 1 and info["sigma"] == [1] and (d.cpu().numpy() == x).all()
    # A X + X A: every sum here has at most 4 terms of under 30 bits and is exact
    p = (np.arange(n) + half) % n
    z = 0.5 * (a - a[:, p]) + 0.5 * (a - a[p, :])
    got, want = chi.cpu().numpy(), (-z).astype(np.float32)
    assert (got == want).all(), (int((got != want).sum()), float(np.abs(got - want).max()))

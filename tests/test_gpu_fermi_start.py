"""FP16 split at finite temperature with many doublings: the start E_0 is then tiny
and its copy's smallest step decides the error of D.  The copies of E stand at
2^15, with a step of 2^-39 (FP16's smallest, 2^-24, over 2^15): a rounding error of
2^-39 / sqrt(12) an entry, doubled by each of the m steps that follow, and the
copies of E_1, E_2, ... add halves, quarters, ... of it: for m = 24
2^-15 / sqrt(12) x sqrt(4 / 3) = 1.02e-5 an entry of D (a little less where the
tanh bends).  A copy of E_0 at 2^14 would give 1.83e-5.  Other errors (FP32
accumulation, the split of R) are about 3e-7."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [200, 333])
def test_step_of_the_start(gpu, n):
    import torch

    import paper_2409_17033_amd as dm
    rng = np.random.default_rng(n)
    h = rng.normal(size=(n, n)) / np.sqrt(2 * n)
    h = (h + h.T).astype(np.float32)                    # spectrum within about [-1.5, 1.5]
    kt = 1.5
    w, v = np.linalg.eigh(h.astype(np.float64))
    ref = (v / (1 + np.exp(w / kt))) @ v.T
    _, d, _, info = dm.susceptibility_fermi(torch.from_numpy(h).to(gpu), None, n // 2, kt, canonical=False, mu=0.0,
                                            doublings=24, precision="split_fp16")
    err = np.linalg.norm(d.double().cpu().numpy() - ref) / n
    print(f"\nn = {n}: {err:.2e} an entry, {info['doublings']} doublings")
    assert err <= 1.3e-5

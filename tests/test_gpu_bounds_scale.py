"""H in units of any power of two: the bounds scale with it exactly and D keeps its
bits, up to entries near the largest finite FP32 value (every step of the bounds
and of X_1 = alpha I + beta H scales exactly; the entries' norm is above 1, where
the search's tolerance is relative)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [8, 32])
@pytest.mark.parametrize("n", [40, 128, 200, 1000])
def test_bounds_in_any_unit(gpu, n, steps):
    import torch

    import paper_2409_17033_amd as dm
    rng = np.random.default_rng(n)
    h = rng.normal(size=(n, n)) / np.sqrt(n)
    h = (h + h.T + np.diag(rng.uniform(-2, 2, n))).astype(np.float32)
    h = np.triu(h) + np.triu(h, 1).T
    H = torch.from_numpy(h).to(gpu)
    D, ref = dm.sp2_density(H, n // 2, lanczos_steps=steps, raise_on_error=False)
    for k in (60, 115, 122):
        Dk, info = dm.sp2_density((H * 2.0 ** k).contiguous(), n // 2, lanczos_steps=steps, raise_on_error=False)
        assert np.ldexp(info["emin"], -k) == pytest.approx(ref["emin"], rel=1e-12)
        assert np.ldexp(info["emax"], -k) == pytest.approx(ref["emax"], rel=1e-12)
        assert info["m"] == ref["m"] and torch.equal(Dk, D)

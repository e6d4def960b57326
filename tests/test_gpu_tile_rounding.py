"""FP32 errors of D at a size where one observable runs on 32 x 32 tiles and four
on 64 x 64 ones: both accumulate in FP32 chains of 64 columns, so they have the same
rounding error as long as the chains end alike with respect to the tile's own rows
and columns (whose terms are the largest).  The error norms are over 5e5 entries; the
bound of 1.12 leaves room for steps whose sigma differs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [640, 760])
def test_tile_edge_does_not_change_the_error(gpu, n):
    import torch

    import paper_2409_17033_amd as dm
    errs = np.zeros((2, 4))
    for seed in range(4):
        rng = np.random.default_rng([n, seed])
        nocc = int((0.3 + 0.1 * seed) * n)
        w = np.sort(rng.uniform(-1.75, 1.75, n))
        w[:nocc] -= 0.05
        w[nocc:] += 0.05
        h = np.diag(w)
        for u in rng.normal(size=(3, n)):          # three reflections on both sides
            u /= np.linalg.norm(u)
            h = h - 2 * np.outer(u, u @ h)
            h = h - 2 * np.outer(h @ u, u)
        h = (0.5 * (h + h.T)).astype(np.float32)
        _, v = np.linalg.eigh(h.astype(np.float64))
        ref = v[:, :nocc] @ v[:, :nocc].T
        a = rng.normal(size=(4, n, n)).astype(np.float32)
        a = a + a.transpose(0, 2, 1)
        H, A = torch.from_numpy(h).to(gpu), torch.from_numpy(a).to(gpu)
        for q, k in enumerate((1, 4)):
            d = dm.susceptibility(H, A[:k], nocc)[1]
            errs[q, seed] = np.linalg.norm(d.double().cpu().numpy() - ref)
    print(f"\nn = {n}: 32 x 32 {errs[0]}, 64 x 64 {errs[1]}")
    assert errs[0].mean() <= 1.12 * errs[1].mean()

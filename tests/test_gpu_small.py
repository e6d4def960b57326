"""Small-size kernels at the edges of their tiles and dispatch.

Partial recursions (five steps, no projection) on two observables against the
FP64 recursion on the sigma sequence and bounds the device chose, with the
per-step bounds that the large-size kernels are held to (2e-6 a step for the
FP32-accurate products, 6e-5 where the sweep products have two BF16 terms).
Sizes: one partial tile of 32, whole tiles and one row more, an odd number of
64-row blocks, the first sizes of the 64 x 64 tiles, a tile count just above
the number of CUs (eight waves a tile), and the last size of the wide-list rule.
"""
import numpy as np
import pytest

import workloads as W
from oracle import closed_form as cf
from oracle import sp2

pytestmark = pytest.mark.gpu

STEPS = 5


@pytest.fixture(scope="module")
def inputs():
    cache = {}

    def get(n):
        if n not in cache:
            wl = W.dense_gapped(n, nocc=max(1, n // 3), nobs=2, npert=1, cfg=21)
            cache[n] = wl
        return cache[n]
    return get


@pytest.mark.parametrize("prec", ["fp32", "split_fp16", "split3_bf16", "split3x_bf16", "split_bf16"])
@pytest.mark.parametrize("n", [5, 32, 33, 64, 95, 129, 449, 705, 960, 1030])
def test_partial_recursion_at_tile_edges(gpu, inputs, n, prec):
    import torch

    import paper_2409_17033_amd as dm
    wl = inputs(n)
    H, A = torch.from_numpy(wl.H).to(gpu), torch.from_numpy(wl.A).to(gpu)
    chi, D, _, info = dm.susceptibility(H, A, wl.nocc, precision=prec, bounds="gershgorin", max_iter=STEPS,
                                        min_iter=STEPS + 1, project=False, spin=1.0, raise_on_error=False)
    assert info["m"] == STEPS and info["tile"] in (32, 64)
    h = wl.H.astype(np.float64)
    xs, beta = sp2.sp2_sequence(h, info["sigma"], info["emin"], info["emax"])
    tol = 6e-5 * STEPS if prec in ("split_bf16", "split3x_bf16") else 2e-6 * STEPS
    assert cf.rel_frobenius(D.double().cpu().numpy(), xs[-1]) < tol
    for k in range(2):
        y = sp2.forward_sweep(xs, info["sigma"], beta, wl.A[k].astype(np.float64))
        c = chi[k].double().cpu().numpy()
        assert cf.rel_frobenius(c, y) < tol
        assert np.array_equal(c, c.T)


@pytest.mark.parametrize("prec,n,tile", [("fp32", 800, 64), ("split_fp16", 800, 32), ("split_fp16", 850, 64),
                                         ("fp32", 900, 32), ("fp32", 960, 32), ("fp32", 961, 64)])
def test_tile_choice_around_one_round(gpu, inputs, prec, n, tile):
    """The sizes where the tile edge and the waves of a workgroup change (two
    observables; FP32 at n = 800: eight waves)."""
    import torch

    import paper_2409_17033_amd as dm
    wl = inputs(n)
    H, A = torch.from_numpy(wl.H).to(gpu), torch.from_numpy(wl.A).to(gpu)
    chi, D, _, info = dm.susceptibility(H, A, wl.nocc, precision=prec, bounds="gershgorin", max_iter=STEPS,
                                        min_iter=STEPS + 1, project=False, spin=1.0, raise_on_error=False)
    assert info["m"] == STEPS and info["tile"] == tile
    xs, beta = sp2.sp2_sequence(wl.H.astype(np.float64), info["sigma"], info["emin"], info["emax"])
    assert cf.rel_frobenius(D.double().cpu().numpy(), xs[-1]) < 2e-6 * STEPS
    for k in range(2):
        y = sp2.forward_sweep(xs, info["sigma"], beta, wl.A[k].astype(np.float64))
        assert cf.rel_frobenius(chi[k].double().cpu().numpy(), y) < 2e-6 * STEPS


@pytest.mark.parametrize("prec,n,nobs", [("fp32", 1985, 1), ("fp32", 2048, 1), ("fp32", 2112, 1), ("fp32", 2240, 1),
                                         ("split_fp16", 2048, 1), ("split_fp16", 2112, 1), ("split3_bf16", 2048, 1),
                                         ("fp32", 1440, 2)])
def test_tiles_in_quarters(gpu, inputs, prec, n, nobs):
    """Sizes whose last tiles run as quarters in the launches of one kind (the
    adjoint solve, which sweeps only after a converged recursion) or of both (the
    partial forward recursion), against the FP64 recursion on the device."""
    import torch

    import paper_2409_17033_amd as dm
    wl = inputs(n)
    H, A = torch.from_numpy(wl.H).to(gpu), torch.from_numpy(wl.A[:nobs]).to(gpu)
    eye = torch.eye(n, dtype=torch.float64, device=gpu)

    def step(y, x, s):
        z = torch.stack([yk @ x for yk in y])
        z = z + z.transpose(1, 2)
        return z if s > 0 else 2 * y - z

    for kw in ({"max_iter": STEPS, "min_iter": STEPS + 1, "raise_on_error": False}, {"sweep": "adjoint"}):
        chi, D, _, info = dm.susceptibility(H, A, wl.nocc, precision=prec, bounds="gershgorin", project=False, spin=1.0,
                                            **kw)
        assert info["tile"] == 64
        m = info["m"]
        beta = 1.0 / (info["emax"] - info["emin"])
        xs = [beta * (info["emax"] * eye - H.double())]
        for s in info["sigma"][:m]:
            xs.append(xs[-1] @ xs[-1] if s > 0 else 2 * xs[-1] - xs[-1] @ xs[-1])
        y = -beta * A.double()
        order = range(m) if "max_iter" in kw else range(m - 1, -1, -1)
        for q in order:
            y = step(y, xs[q], info["sigma"][q])
        assert float((D.double() - xs[m]).norm() / xs[m].norm()) < 2e-6 * m
        for k in range(nobs):
            assert float((chi[k].double() - y[k]).norm() / y[k].norm()) < 2e-6 * m
            assert torch.equal(chi[k], chi[k].T)


@pytest.mark.parametrize("prec", ["fp32", "split_fp16", "split3x_bf16"])
@pytest.mark.parametrize("n", [31, 64, 100, 500, 512, 700, 1000, 1024])
def test_diagonal_tiles_of_one_observable(gpu, inputs, n, prec):
    """One observable: Z's diagonal tiles from one product and its transpose, in
    the order that spreads them (fewer than 16 tile rows: all of them last)."""
    import torch

    import paper_2409_17033_amd as dm
    wl = inputs(n)
    H, A = torch.from_numpy(wl.H).to(gpu), torch.from_numpy(wl.A[0]).to(gpu)
    chi, D, _, info = dm.susceptibility(H, A, wl.nocc, precision=prec, bounds="gershgorin", max_iter=STEPS,
                                        min_iter=STEPS + 1, project=False, spin=1.0, raise_on_error=False)
    assert info["m"] == STEPS and info["tile"] in (32, 64)
    xs, beta = sp2.sp2_sequence(wl.H.astype(np.float64), info["sigma"], info["emin"], info["emax"])
    tol = 6e-5 * STEPS if prec == "split3x_bf16" else 2e-6 * STEPS
    c = chi.double().cpu().numpy()
    y = sp2.forward_sweep(xs, info["sigma"], beta, wl.A[0].astype(np.float64))
    assert cf.rel_frobenius(D.double().cpu().numpy(), xs[-1]) < tol
    assert cf.rel_frobenius(c, y) < tol and np.array_equal(c, c.T)


@pytest.mark.parametrize("n,tile", [(1984, 64), (1985, 256)])
def test_wide_list_runs_keep_the_large_tiles(gpu, n, tile):
    """Corrected runs of the three-term-X^2 option change to the large-size
    lists above n = 1984; both sides meet the refined 1e-5."""
    import torch

    import paper_2409_17033_amd as dm
    wl = W.banded_gapped(n, cfg=22, npert=1, cache=False)
    chi, D, _, info = dm.susceptibility(torch.from_numpy(wl.H).to(gpu), torch.from_numpy(wl.A[0]).to(gpu), wl.nocc,
                                        precision="split3x_bf16", refine=True, sweep_tol=1e-3)
    assert info["tile"] == tile
    ref = cf.susceptibility(wl.H.astype(np.float64), wl.A[0].astype(np.float64), wl.nocc, spin=2.0)
    assert cf.rel_frobenius(chi.double().cpu().numpy(), ref) <= 1e-5

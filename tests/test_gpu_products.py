"""General products (the finite-temperature recursion) at the edges of their
tiles, job lists and batches, against the same recursion in FP64 with exact
inverses.

Eight doublings to beta w = 12.8 at a given mu (the start is then linear to
beta w / 2^8 = 0.05 in both).  Bound: 2e-6 a doubling for products of FP32
accuracy (five products each, the relative error of E and Y does not grow
through a doubling), 6e-5 where operands have two BF16 terms, as for the steps of
the zero-temperature recursion.  Sizes: one partial tile, whole tiles and a
row more, an odd number of 64-row blocks, the change to 64 x 64 tiles, the last
size of the square tiles and the first of the large ones (tiles in pieces of
their K range), for each precision; batches with a remainder in the last group.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

M, BW = 8, 12.8


def _inputs(n, nobs, gpu):
    import torch
    rng = np.random.default_rng(100 + n)
    h = torch.from_numpy(rng.standard_normal((n, n)).astype(np.float32)).to(gpu)
    h = ((h + h.T) / (2.0 * (2.0 * n) ** 0.5)).contiguous()       # spectrum about [-1, 1]
    a = torch.from_numpy(rng.standard_normal((nobs, n, n)).astype(np.float32)).to(gpu)
    return h, ((a + a.transpose(1, 2)) / 2).contiguous()


def _solve(h, a, kt, mu, prec):
    import paper_2409_17033_amd as dm
    return dm.susceptibility_fermi(h, a, h.shape[0] // 2, kt, canonical=False, mu=mu, doublings=M,
                                   bounds="gershgorin", precision=prec, spin=1.0)


def _reference(h, a, kt, mu):
    import torch
    n = h.shape[0]
    eye = torch.eye(n, dtype=torch.float64, device=h.device)
    c = 1.0 / kt / 2.0 ** (M + 2)
    e, y = c * (mu * eye - h.double()), -c * a.double()
    for _ in range(M):
        r = torch.linalg.inv(eye + 4.0 * e @ e)
        en = 2.0 * e @ r
        for k in range(a.shape[0]):
            s = y[k] @ e + e @ y[k]
            w = (2.0 * y[k] - 4.0 * en @ s) @ r
            y[k] = (w + w.T) / 2
        e = (en + en.T) / 2
    return 0.5 * eye + e, y


@pytest.mark.parametrize("prec,n,nobs", [
    *((p, n, 2) for p in ("fp32", "split_fp16", "split3_bf16", "split_bf16") for n in (5, 33, 64, 129, 1030)),
    ("fp32", 1600, 1), ("split_fp16", 700, 1), ("split_fp16", 2100, 17),
    ("split_fp16", 2944, 2), ("split_fp16", 2945, 5), ("split3_bf16", 2945, 1), ("split_bf16", 2945, 1),
    ("fp32", 3328, 1), ("fp32", 3329, 2), ("split_fp16", 4096, 1)])
def test_recursion_at_tile_and_list_edges(gpu, prec, n, nobs):
    import torch
    h, a = _inputs(n, nobs, gpu)
    w = float(h.abs().sum(1).max())
    kt, mu = w / BW, 0.05 * w
    chi, D, a0, info = _solve(h, a, kt, mu, prec)
    d_ref, y_ref = _reference(h, a, kt, mu)
    tol = M * (6e-5 if prec == "split_bf16" else 2e-6)
    err_d = float((D.double() - d_ref).norm() / d_ref.norm())
    err_y = max(float((chi[k].double() - y_ref[k]).norm() / y_ref[k].norm()) for k in range(nobs))
    print(f"\n{prec} n={n}: errD {err_d:.2e} errY {err_y:.2e}")
    assert info["doublings"] == M and err_d < tol and err_y < tol
    assert torch.equal(D, D.T) and all(torch.equal(chi[k], chi[k].T) for k in range(nobs))
    one, _, _, _ = _solve(h, a[nobs - 1].contiguous(), kt, mu, prec)
    assert torch.equal(one, chi[nobs - 1])

"""Rank-k updates C + X Y^H at the edges of the real form's 64 x 32 tiles, which
take C ahead of the products: odd orders around the 1024 tiles of 32 x 32 where
it begins (n = 993) and ranks around the 448 where it ends, alone and two in
one pass.

Tolerance: k products and the sums of an entry round by at most (k + 4) u of
its terms' magnitudes (u = 2^-53), with a factor 2 for the scaled factor."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def _randn(n, k, dt, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(n, k, dtype=dt, device="cuda", generator=g)


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("n,k", [(991, 3), (993, 1), (993, 2), (1023, 33), (1025, 16), (1057, 97),
                                 (1025, 447), (1025, 448), (1025, 449), (2081, 40)])
def test_one_update(cplx, n, k):
    import torch
    import paper_2205_02491_amd as pk
    announce(f"rank-{k} update of order {n} cplx={cplx}")
    dt = torch.complex128 if cplx else torch.float64
    v, d0 = _randn(n, k, dt, n + k), _randn(n, n, dt, n)
    g = np.random.Generator(np.random.PCG64(k)).standard_normal(k)
    dh = d0.clone()
    pk.chase_eigval_adjoint(v, g, dh)
    gt = torch.from_numpy(g).cuda()
    ref = d0 + torch.matmul(v * gt, v.mH.contiguous())
    lim = 2 * (k + 4) * U * (d0.abs() + torch.matmul(v.abs() * gt.abs(), v.abs().mT.contiguous()))
    # the reference rounds as much
    assert bool(((dh - ref).abs() <= 2 * lim).all())


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("n,k", [(991, 5), (993, 7), (1025, 33), (1057, 200)])
def test_two_updates_in_one_pass(cplx, n, k):
    """The filter adjoint of degrees 2 and 4: its pairs of updates have ranks
    that differ.  Reference: torch's autograd of the recurrence in FP64; six
    products of length n and the sums over k columns."""
    import torch
    import paper_2205_02491_amd as pk
    announce(f"pairs of rank-k updates n={n} k={k} cplx={cplx}")
    dt = torch.complex128 if cplx else torch.float64
    z = _randn(n, n, dt, 3 * n)
    H = (z + z.mH) / (2.0 * (2.0 * n) ** 0.5)
    X, gY = _randn(n, k, dt, n + 1), _randn(n, k, dt, n + 2)
    deg = np.where(np.arange(k) < k // 3, 2, 4).astype(np.int32)
    b_sup, mu_1, mu_ne = 1.05, -1.02, -0.5
    coef = pk.chase_filter_coefficients(4, b_sup, mu_1, mu_ne).reshape(4, 3)
    with pk.Handle(n, k - 1, 1, dt, pk.default_opts(adjoint_reserve=4)) as hd:
        pk.chase_filter(H, X, deg, b_sup, mu_1, mu_ne, record_tape=True, handle=hd)
        dH = torch.zeros_like(H)
        gX = pk.chase_filter_adjoint(H, gY, dH, hd, want_gX=True)
    Ht, Xt = H.clone().requires_grad_(True), X.clone().requires_grad_(True)
    prev, cur, out = torch.zeros_like(Xt), Xt, torch.zeros_like(Xt)
    for s, (a, c, b) in enumerate(coef, 1):
        prev, cur = cur, a * (torch.matmul(Ht, cur) - c * cur) + b * prev
        out = torch.where(torch.from_numpy(deg == s).cuda()[None, :], cur, out)
    rH, rX = torch.autograd.grad(out, (Ht, Xt), gY)
    rH = (rH + rH.mH) / 2
    tol = 100 * (n + k) * U
    assert float((dH - rH).abs().max()) <= tol * float(rH.abs().max())
    assert float((gX - rX).abs().max()) <= tol * float(rX.abs().max())

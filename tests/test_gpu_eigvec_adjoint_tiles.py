"""The eigenvector adjoint's shifted products (H - lambda_j) p_j over the tiles
that the products with H take: a single column, ragged orders and blocks, and a
block that fills the chip with large tiles.

Reference: first-order perturbation on the planted eigenvectors.  The gap below
the other eigenvalues is 0.3 and |H| = 1, so conjugate gradients stopped at
1e-11 of the first residual leave at most 1e-11 / 0.3 of a column, times
sqrt(m) over the block, and the planted vectors are off by n u / 0.3: 1e-9 of
the gradient's largest entry."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("n,m", [(17, 1), (97, 5), (259, 33), (1101, 129), (2047, 65), (1500, 501)])
def test_shifted_products(cplx, n, m):
    import torch
    import paper_2205_02491_amd as pk
    announce(f"eigenvector adjoint n={n} m={m} cplx={cplx}")
    dt = torch.complex128 if cplx else torch.float64
    g = torch.Generator(device="cuda").manual_seed(71 * n + m)
    q, r = torch.linalg.qr(torch.randn(n, n, dtype=dt, device="cuda", generator=g))
    lam = torch.cat([torch.linspace(-1.0, -0.8, m, dtype=torch.float64),
                     torch.linspace(-0.5, 1.0, n - m, dtype=torch.float64)]).cuda()
    h = torch.matmul(q * lam, q.mH.contiguous())
    h = ((h + h.mH) / 2).contiguous()
    v, gv = q[:, :m].contiguous(), torch.randn(n, m, dtype=dt, device="cuda", generator=g)
    dh = torch.zeros_like(h)
    pk.chase_eigvec_adjoint(h, v, lam[:m].cpu().numpy(), gv, dh, tol=1e-11)
    c = torch.matmul(q.mH, gv)
    den = lam[None, :m] - lam[:, None]
    same = torch.arange(m, device="cuda")
    den[same, same] = 1.0
    f = c / den.to(dt)
    f[same, same] = 0.0
    a = torch.matmul(torch.matmul(q, f), v.mH.contiguous())
    ref = (a + a.mH) / 2
    assert float((dh - ref).abs().max()) <= 1e-9 * float(ref.abs().max())

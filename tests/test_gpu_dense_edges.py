"""Edges of the k x k kernels: the Jacobi rounds at block counts where pairs,
padding and the eigenvector tiles change, its sort on repeated eigenvalues,
and the Cholesky QR on both sides of the order (512) up to which one launch
inverts the factor.

Tolerances.  Jacobi stops at an off-diagonal norm of 1e-14 |G|_F (|G|_F <= 10
here: 1e-13) and rounds by a few u |G|_F in each of at most 200 rounds (2e-13):
1e-12 on residual and orthonormality, per column.  QR: k u times a small
constant per entry of Q^H Q: 1e-13 sqrt(k) in the Frobenius norm, and 1e-11
on the projector onto the block's span (condition 10 k)."""
import numpy as np
import pytest

import gen
import oracle
from gpu_util import announce, to_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pk():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2205_02491_amd as pk
    pk.lib()
    return pk


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("k", [1, 2, 16, 31, 33, 48, 49, 64, 65, 97])
def test_jacobi_rounds_and_repeated_eigenvalues(pk, cplx, k):
    announce(f"Jacobi rounds k={k} cplx={cplx}")
    g = np.random.Generator(np.random.PCG64(53 * k + cplx))
    q = np.linalg.qr(gen.gaussian(g, (k, k), cplx))[0]
    lam = np.repeat(np.linspace(-1.0, 1.0, (k + 2) // 3), 3)[:k]  # triples
    a = (q * lam) @ q.conj().T
    for m in ((a + a.conj().T) / 2, np.diag(lam[::-1]).astype(q.dtype), np.zeros_like(q)):
        w, v, _ = pk.chase_heev(to_gpu(m), pk.EIG_JACOBI)
        v = to_np(v)
        assert np.all(np.diff(w) >= 0)
        assert np.max(np.abs(w - np.linalg.eigvalsh(m))) < 1e-12
        assert np.max(np.linalg.norm(m @ v - v * w, axis=0)) < 1e-12
        assert np.max(np.linalg.norm(v.conj().T @ v - np.eye(k), axis=0)) < 1e-12


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,k,locked", [(40, 1, 0), (70, 31, 0), (70, 32, 5), (90, 33, 0),
                                        (300, 256, 0), (300, 257, 40), (700, 511, 0),
                                        (700, 512, 0), (700, 513, 0), (700, 600, 90)])
def test_qr_inverse_orders(pk, cplx, n, k, locked):
    announce(f"QR n={n} k={k} locked={locked} cplx={cplx}")
    g = np.random.Generator(np.random.PCG64(59 * n + k))
    x = gen.gaussian(g, (n, k), cplx) * np.logspace(0, 1, k)
    if locked:
        x[:, :locked] = np.linalg.qr(x[:, :locked])[0]
    ref = np.linalg.qr(x)[0]
    q = to_np(pk.chase_qr(to_gpu(x), locked))
    assert np.array_equal(q[:, :locked], x[:, :locked])
    assert np.linalg.norm(q.conj().T @ q - np.eye(k)) < 1e-13 * max(1.0, np.sqrt(k))
    assert np.linalg.norm(q - ref @ (ref.conj().T @ q)) < 1e-11


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,deg", [(2, (2,)), (31, (2, 2, 4, 8)), (32, (6,) * 5),
                                   (33, (2, 4, 4, 10, 12)), (65, (4,) * 3 + (6,) * 30),
                                   (130, (2, 14)), (993, (2,) * 3 + (4,) * 30),
                                   (1025, (2, 4, 6, 6, 8)), (1060, (2,) * 180 + (4,) * 20)])
def test_filter_adjoint_edges(pk, cplx, n, deg):
    """Reverse sweep with columns that join it at different steps, the rank-k
    updates of two steps in one pass (from order 993; the real one up to 192
    columns) and the Hermitian part at tile edges (32), against automatic differentiation of
    the recurrence on the CPU.  Both sides round n u per product and amplify
    by less than 4 s per step (s <= 14): 1e-11 of the largest entry."""
    import torch
    announce(f"filter adjoint edges n={n} deg={deg} cplx={cplx}")
    g = np.random.Generator(np.random.PCG64(61 * n + len(deg)))
    k = len(deg)
    z = gen.gaussian(g, (n, n), cplx)
    z = z + z.conj().T
    z /= np.linalg.norm(z, 2)
    x0, gy = gen.gaussian(g, (n, k), cplx), gen.gaussian(g, (n, k), cplx)
    b_sup, mu_1, mu_ne = 1.05, -1.02, -0.5

    hc, xc = torch.from_numpy(z).requires_grad_(True), torch.from_numpy(x0).requires_grad_(True)
    c, e = (b_sup + mu_ne) / 2, (b_sup - mu_ne) / 2
    hs = hc - c * torch.eye(n, dtype=hc.dtype)
    s1 = e / (mu_1 - c)
    prev, cur, sig = xc, (s1 / e) * (hs @ xc), s1
    cols = [None] * k
    for s in range(2, deg[-1] + 1):
        sn = 1.0 / (2.0 / s1 - sig)
        prev, cur = cur, (2.0 * sn / e) * (hs @ cur) - sig * sn * prev
        sig = sn
        for a in range(k):
            if deg[a] == s:
                cols[a] = cur[:, a]
    yc = torch.stack(cols, dim=1)
    torch.sum(torch.real(torch.conj(torch.from_numpy(gy)) * yc)).backward()
    dh_ref = hc.grad.numpy()
    dh_ref = (dh_ref + dh_ref.conj().T) / 2

    h, x = to_gpu(z).requires_grad_(True), to_gpu(x0).requires_grad_(True)
    y = pk.filtered_block(h, x, np.array(deg, np.int32), b_sup, mu_1, mu_ne)
    torch.sum(torch.real(torch.conj(to_gpu(gy)) * y)).backward()
    for got, ref in ((y.detach(), yc.detach().numpy()), (h.grad, dh_ref),
                     (x.grad, xc.grad.numpy())):
        assert np.max(np.abs(to_np(got) - ref)) <= 1e-11 * np.max(np.abs(ref))
    dh = to_np(h.grad)
    assert np.array_equal(dh, dh.conj().T)


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,m", [(40, 3), (1000, 1), (1000, 33), (1031, 195)])
def test_eigvec_adjoint_rank_updates(pk, cplx, n, m):
    """Eigenvector adjoint, whose two rank-m updates run in one pass from
    order 993 (the real one up to 192 columns), against the oracle's
    first-order perturbation.  Conjugate gradients to 1e-12 across a gap of
    0.3, divided differences of rounding (1e-13) over gaps of 1 / (5 m) >=
    1e-3: 1e-8 of the norm."""
    import torch
    announce(f"eigvec adjoint rank updates n={n} m={m} cplx={cplx}")
    g = np.random.Generator(np.random.PCG64(67 * n + m))
    q = np.linalg.qr(gen.gaussian(g, (n, n), cplx))[0]
    lam = np.concatenate([-1.0 + 0.25 * (np.arange(m) + g.uniform(0.0, 0.2, m)) / m,
                          np.linspace(-0.45, 1.0, n - m)])
    h = (q * lam) @ q.conj().T
    h = (h + h.conj().T) / 2
    v, gv = q[:, :m].copy(), gen.gaussian(g, (n, m), cplx)
    ref = oracle.eigvec_adjoint(h, v, lam[:m], gv)
    dh = torch.zeros((n, n), dtype=to_gpu(h).dtype, device="cuda")
    pk.chase_eigvec_adjoint(to_gpu(h), to_gpu(v), lam[:m], to_gpu(gv), dh, tol=1e-12)
    assert np.linalg.norm(to_np(dh) - ref) <= 1e-8 * np.linalg.norm(ref)

"""Columns further apart than their length, blocks that begin inside a buffer:
FP32 filter steps (whose kernel depends on where the columns of H and of the
block lie), the adjoints' rank-k updates and shifted products, and Lanczos give
what they give on closely packed columns, and write nothing between them.

Tolerances.  Against packed columns: FP32 steps round with random sign, 2^-24
sqrt(n) of a column's size, 16 times that for two steps of two runs and the
largest entry.  A rank-k update sums k products: 8 (k + 8) u of the magnitudes.
The linear solves stop at residuals of 1e-12 over a gap of 0.9 in the spectrum:
two of them are within 1e-11 of the largest entry times sqrt(n) <= 40.  Lanczos:
six steps of the recurrence, 2^6 n u < 1e-11."""
import ctypes

import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu
U = 2.0 ** -53
MARK = 7.75


class Block:
    """An n x k block in a marked buffer, columns `ld` apart, first at `off`."""

    def __init__(self, data, pad=0, off=0):
        import torch
        n, k = data.shape
        self.ld = n + pad
        self.shape, self.strides, self.off = (n, k), (1, self.ld), off
        self.buf = torch.full((off + self.ld * k + 3,), MARK, dtype=data.dtype, device="cuda")
        self.view.copy_(data)
        self.ptr = self.buf.data_ptr() + off * self.buf.element_size()

    @property
    def view(self):
        import torch
        return torch.as_strided(self.buf, self.shape, self.strides, self.off)

    def result(self):
        import torch
        out = self.view.clone()
        self.view.fill_(MARK)
        assert bool((self.buf == MARK).all()), "written outside the block"
        return out


def _rnd(n, k, cplx, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn(n, k, dtype=torch.complex128 if cplx else torch.float64, device="cuda",
                       generator=g)


def _herm(n, cplx):
    z = _rnd(n, n, cplx, n)
    return z.add(z.mH).div_(2.0 * (2.0 * n) ** 0.5)


def _p(a):
    return a.ctypes.data_as(ctypes.POINTER(ctypes.c_double))


def _handle(pk, n, k, x, **opts):
    return pk.Handle(n, max(1, k - 1), 1, x.dtype, pk.default_opts(**opts))


# (n, k, complex, handle holds H in FP32): the packed columns of the orders that are
# multiples of 8 lie on the cache lines, padded ones off them, which changes the tile
# table and, for the wide blocks, lets the staged kernel in
FP32 = [(3000, 1900, False, True), (3000, 1900, False, False), (8000, 704, False, False),
        (9600, 736, True, True), (9600, 736, True, False), (640, 40, True, True),
        (1001, 37, False, True), (1001, 37, False, False), (17, 3, True, False)]


@pytest.mark.parametrize("n,k,cplx,copy", FP32)
def test_fp32_steps(n, k, cplx, copy):
    import paper_2205_02491_amd as pk
    L = pk.lib()
    h, x = _herm(n, cplx), _rnd(n, k, cplx, 3)
    d = np.full(k, 2, np.int32)
    opts = dict(filter_prec=pk.PREC_FP32) if copy else {}
    ref = None
    for hp, ho, xp, xo in [(0, 0, 0, 0), (1, 0, 0, 0), (0, 0, 3, 1), (7, 1, 1, 3)]:
        announce(f"leading dims: FP32 n={n} k={k} cplx={cplx} copy={copy} pads {hp},{ho} {xp},{xo}")
        H, X = Block(h, hp, ho), Block(x, xp, xo)
        with _handle(pk, n, k, x, **opts) as hd:
            pk._check(L.chase_filter(hd.ptr, H.ptr, H.ld, X.ptr, X.ld, k,
                                     d.ctypes.data_as(ctypes.POINTER(ctypes.c_int)), 1.05, -1.02,
                                     -0.5, pk.PREC_FP32, 0, None, None))
        H.result()
        out = X.result()
        if ref is None:
            ref, lim = out, 16 * 2.0 ** -24 * n ** 0.5 * out.abs().amax(0)
        assert bool(((out - ref).abs().amax(0) <= lim).all())


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,k", [(1200, 60), (1025, 449), (1024, 448), (63, 5)])
def test_rank_updates(cplx, n, k):
    import torch
    import paper_2205_02491_amd as pk
    L = pk.lib()
    v, d0 = _rnd(n, k, cplx, 4), _herm(n, cplx)
    g = np.linspace(-1.0, 2.0, k)
    gt = torch.from_numpy(g).cuda()
    mag = d0.abs() + torch.matmul(v.abs() * gt.abs(), v.abs().T.contiguous())
    ref = None
    for vp, vo, dp, do in [(0, 0, 0, 0), (1, 1, 3, 1), (5, 0, 0, 3)]:
        announce(f"leading dims: rank n={n} k={k} cplx={cplx} pads {vp},{vo} {dp},{do}")
        V, D = Block(v, vp, vo), Block(d0, dp, do)
        with _handle(pk, n, k, v) as hd:
            pk._check(L.chase_eigval_adjoint(hd.ptr, V.ptr, V.ld, k, _p(g), D.ptr, D.ld, None))
        V.result()
        out = D.result()
        ref = out if ref is None else ref
        assert bool(((out - ref).abs() <= 8 * (k + 8) * U * mag).all())


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,k", [(1000, 33), (517, 96), (64, 4)])
def test_shifted_products(cplx, n, k):
    import torch
    import paper_2205_02491_amd as pk
    L = pk.lib()
    q = torch.linalg.qr(_rnd(n, n, cplx, 5))[0]
    lam = torch.cat([torch.linspace(-1.0, -0.9, k, dtype=torch.float64),
                     torch.linspace(0.0, 1.0, n - k, dtype=torch.float64)]).cuda()
    h = torch.matmul(q * lam, q.mH.contiguous())
    h = h.add(h.mH).div_(2.0)
    lh = lam[:k].cpu().numpy()
    gy, zero = _rnd(n, k, cplx, 6), torch.zeros_like(h)
    ref = None
    for hp, ho, vp, vo in [(0, 0, 0, 0), (1, 1, 3, 0), (3, 0, 0, 1)]:
        announce(f"leading dims: eigvec n={n} k={k} cplx={cplx} pads {hp},{ho} {vp},{vo}")
        H, V = Block(h, hp, ho), Block(q[:, :k], vp, vo)
        G, D = Block(gy, vo, vp), Block(zero, hp, ho)
        it = ctypes.c_int()
        with _handle(pk, n, k, h) as hd:
            pk._check(L.chase_eigvec_adjoint(hd.ptr, H.ptr, H.ld, V.ptr, V.ld, k, _p(lh), G.ptr,
                                             G.ld, D.ptr, D.ld, 1e-12, 500, ctypes.byref(it), None))
        for b in (H, V, G):
            b.result()
        out = D.result()
        ref = out if ref is None else ref
        assert float((out - ref).abs().max()) <= 4e-10 * float(ref.abs().max())


@pytest.mark.parametrize("n,cplx", [(2199, True), (2201, True), (2200, False), (4097, False)])
def test_lanczos_products(n, cplx):
    import paper_2205_02491_amd as pk
    L = pk.lib()
    h, s = _herm(n, cplx), _rnd(3, n, cplx, 7)
    ref = None
    for hp, ho in [(0, 0), (1, 0), (3, 1)]:
        announce(f"leading dims: lanczos n={n} cplx={cplx} pads {hp},{ho}")
        H = Block(h, hp, ho)
        a, b, o = np.zeros((3, 6)), np.zeros((3, 6)), [ctypes.c_double() for _ in range(3)]
        with _handle(pk, n, 3, s, lanczos_vecs=3, lanczos_steps=6) as hd:
            pk._check(L.chase_lanczos(hd.ptr, H.ptr, H.ld, s.data_ptr(), 3, 6,
                                      *[ctypes.byref(z) for z in o], _p(a), _p(b), None, None))
        H.result()
        ref = (a, b) if ref is None else ref
        assert max(np.abs(a - ref[0]).max(), np.abs(b - ref[1]).max()) <= 1e-10

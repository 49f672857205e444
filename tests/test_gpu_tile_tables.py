"""Every tile of the products' tables at odd orders and ragged blocks: filter
steps in FP64, FP32 and on INT8, and the short products of QR.  (Which shape
takes which tile is held to the sources by the test without a GPU.)

Tolerances.  FP64: two steps; a product of length n errs by at most (n + 8) u
of its terms' magnitudes, the three-product form by four times that, so 8 (n +
8) u times the recurrence run on magnitudes covers both steps, entry by entry.
FP32: rounding errors of random sign, 2^-24 sqrt(n) of a column's size in each
step; 16 times that for both steps and the largest of up to 8e6 entries, where
one lost term of a product would be n^-1/2, hundreds of times more.  INT8: the
FP64 bar of 1e-12 of a column's largest entry (integer forms of 46 bits and
more).  QR: k u times a small constant per entry of Q^H Q."""
import numpy as np
import pytest

import tile_tables as tt
from gpu_util import announce

pytestmark = pytest.mark.gpu
U = 2.0 ** -53
B_SUP, MU_1, MU_NE = 1.05, -1.02, -0.5


def _inputs(n, k, cplx):
    import torch
    dt = torch.complex128 if cplx else torch.float64
    g = torch.Generator(device="cuda").manual_seed(17 * n + k)
    h = torch.randn(n, n, dtype=dt, device="cuda", generator=g)
    h = h.add(h.mH).div_(2.0 * (2.0 * n) ** 0.5)
    return h, torch.randn(n, k, dtype=dt, device="cuda", generator=g)


def _two_steps(pk, h, x, magnitudes=False):
    import torch
    if magnitudes:
        h, x = h.abs(), x.abs()
    prev, cur = torch.zeros_like(x), x
    for a, c, b in pk.chase_filter_coefficients(2, B_SUP, MU_1, MU_NE):
        if magnitudes:
            a, c, b = abs(a), -abs(c), abs(b)
        prev, cur = cur, a * (torch.matmul(h, cur) - c * cur) + b * prev
    return cur


def _filter(pk, h, x, prec, **opts):
    k = x.shape[1]
    with pk.Handle(x.shape[0], k - 1, 1, x.dtype, pk.default_opts(**opts)) as hd:
        return pk.chase_filter(h, x, np.full(k, 2, np.int32), B_SUP, MU_1, MU_NE, prec=prec,
                               handle=hd)[0]


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,k", tt.SHAPES + tt.STAGED_SHAPES)
def test_fp64_and_fp32_tiles(cplx, n, k):
    import paper_2205_02491_amd as pk
    announce(f"tile tables: n={n} k={k} cplx={cplx}")
    h, x = _inputs(n, k, cplx)
    ref = _two_steps(pk, h, x)
    err = (_filter(pk, h, x, pk.PREC_FP64) - ref).abs()
    assert bool((err <= 8 * (n + 8) * U * _two_steps(pk, h, x, True)).all())
    lim = 16 * 2.0 ** -24 * n ** 0.5 * ref.abs().amax(0)
    # with the handle's FP32 copy of H, and rounding H as it is read
    for opts in (dict(filter_prec=pk.PREC_FP32), {}):
        err = (_filter(pk, h, x, pk.PREC_FP32, **opts) - ref).abs().amax(0)
        assert bool((err <= lim).all()), (opts, float((err / lim).max()))


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,k", tt.INT8_SHAPES)
def test_int8_widths(cplx, n, k):
    import paper_2205_02491_amd as pk
    announce(f"tile tables: int8 n={n} k={k} cplx={cplx}")
    h, x = _inputs(n, k, cplx)
    ref = _two_steps(pk, h, x)
    err = (_filter(pk, h, x, pk.PREC_FP64, fp64_emulation=14) - ref).abs().amax(0)
    assert bool((err <= 1e-12 * ref.abs().amax(0)).all())


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,k", [(371, 171), (821, 395), (5001, 201), (8001, 129), (2435, 773)])
def test_short_products_of_qr(cplx, n, k):
    """32 x 32 tiles of two, four and eight waves, 64 x 32 tiles, and the
    Gram matrix's 32 and 64 wide ones."""
    import torch
    import paper_2205_02491_amd as pk
    announce(f"tile tables: QR n={n} k={k} cplx={cplx}")
    x = _inputs(n, k, cplx)[1] * torch.logspace(0, 1, k, dtype=torch.float64, device="cuda")
    q = pk.chase_qr(x)
    eye = torch.eye(k, dtype=x.dtype, device="cuda")
    qh = q.mH.contiguous()
    assert float((torch.matmul(qh, q) - eye).abs().max()) <= 8 * k * U
    assert float((torch.matmul(q, torch.matmul(qh, x)) - x).abs().max()) <= 1e-12 * float(x.abs().max())

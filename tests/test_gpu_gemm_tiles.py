"""Edges of the tile GEMM through the entry points that run it: rows, columns
and K lengths on both sides of the fragment (16), pair (2), stage (4 and 8),
tile (32, 48, 64) and wave-unit boundaries, including a matrix whose columns
are not 16-byte aligned (odd real n).

Tolerances: a product of length n accumulated in FP64 is off by at most
n u |A||B| entrywise (u = 2^-53); the three-product complex form by a small
multiple of it.  Eight filter steps of the scaled recurrence amplify an early
error by less than 4 s per step s, so 1e-12 of a column's largest entry (the
bar of the filter parity test) covers n <= 1100 with degree 8 by more than
an order of magnitude."""
import numpy as np
import pytest

import gen
import oracle
from gpu_util import announce, rel_err, to_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pk():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2205_02491_amd as pk
    pk.lib()
    return pk


def _hermitian(g, n, cplx):
    z = gen.gaussian(g, (n, n), cplx)
    h = (z + z.conj().T) / 2
    return h / np.linalg.norm(h, 2)


SHAPES = [(2, 1), (3, 2), (5, 3), (15, 2), (16, 5), (17, 16), (31, 17), (33, 31), (47, 33),
          (49, 48), (63, 1), (65, 49), (97, 64), (130, 65), (257, 96), (515, 7), (1025, 130)]


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,k", SHAPES)
def test_filter_tile_edges(pk, cplx, n, k):
    announce(f"tile edges: filter n={n} k={k} cplx={cplx}")
    g = np.random.Generator(np.random.PCG64(31 * n + k))
    h, x = _hermitian(g, n, cplx), gen.gaussian(g, (n, k), cplx)
    deg = np.sort(2 * g.integers(1, 5, size=k)).astype(np.int32)
    y_ref, mv_ref = oracle.chebyshev_filter(h, x, deg, 1.05, -1.02, -0.5)
    y, mv = pk.chase_filter(to_gpu(h), to_gpu(x), deg, 1.05, -1.02, -0.5)
    assert mv == mv_ref
    y = to_np(y)
    err = np.max(np.abs(y - y_ref), axis=0) / np.max(np.abs(y_ref), axis=0)
    assert err.max() < 1e-12, (int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,k", [(5, 3), (33, 31), (65, 49), (257, 96), (515, 7)])
def test_filter_fp32_tile_edges(pk, cplx, n, k):
    """FP32 products: the same shapes as a defect-form pass from residuals of
    size 1e-4, whose FP32 rounding (2^-24 sqrt(n) per product, eight steps)
    is relative to the residual: 1e-4 * 1e-5 of the largest entry."""
    announce(f"tile edges: fp32 defect filter n={n} k={k} cplx={cplx}")
    g = np.random.Generator(np.random.PCG64(37 * n + k))
    h = _hermitian(g, n, cplx)
    v = np.linalg.qr(gen.gaussian(g, (n, k), cplx))[0]
    theta = np.linspace(-1.0, -0.6, k)
    r = h @ v - v * theta
    # H' = H - (r v^H + v r^H - v (v^H r) v^H) has H' v = v theta up to a residual
    h2 = h - (1 - 1e-4) * (r @ v.conj().T + v @ r.conj().T - v @ (v.conj().T @ r) @ v.conj().T)
    h2 = (h2 + h2.conj().T) / 2
    r2 = h2 @ v - v * theta
    deg = np.full(k, 8, dtype=np.int32)
    b_sup = 1.05 * max(1.0, np.linalg.norm(h2, 2))
    y_ref, _ = oracle.chebyshev_filter(h2, v, deg, b_sup, -1.02, -0.5)
    y, _ = pk.chase_filter_ritz(to_gpu(h2), to_gpu(v), to_gpu(r2), theta, deg, b_sup, -1.02, -0.5,
                                prec=pk.PREC_FP32)
    assert rel_err(to_np(y), y_ref) < max(1e-9, 1e-5 * np.abs(r2).max() / np.abs(v).max())


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,k", [(3, 2), (17, 16), (33, 31), (65, 49), (259, 97)])
def test_ritz_and_rank_update_tile_edges(pk, cplx, n, k):
    """Projection, Ritz products and residual norms; then the rank-k update
    dH += V diag(g) V^H, entrywise against numpy (k u |V||V| with factor 8)."""
    announce(f"tile edges: Rayleigh-Ritz and rank-k update n={n} k={k} cplx={cplx}")
    g = np.random.Generator(np.random.PCG64(41 * n + k))
    h = _hermitian(g, n, cplx)
    q = np.linalg.qr(gen.gaussian(g, (n, k), cplx))[0]
    ritz, v, res = pk.chase_rayleigh_ritz(to_gpu(h), to_gpu(q))
    v = to_np(v)
    gm = q.conj().T @ h @ q
    assert np.max(np.abs(ritz - np.linalg.eigvalsh((gm + gm.conj().T) / 2))) < 1e-13 * n
    assert np.max(np.abs(v.conj().T @ v - np.eye(k))) < 1e-13 * n
    r_ref = np.linalg.norm(h @ v - v * ritz, axis=0)
    assert np.max(np.abs(res - r_ref)) < 1e-13 * n
    import torch
    gl = g.standard_normal(k)
    d0 = gen.gaussian(g, (n, n), cplx)
    dh = to_gpu(d0).clone()
    pk.chase_eigval_adjoint(torch.from_numpy(np.ascontiguousarray(v)).cuda(), gl, dh)
    ref = d0 + (v * gl) @ v.conj().T
    lim = 8 * (k + 2) * 2.0 ** -53 * (np.abs(d0) + (np.abs(v) * np.abs(gl)) @ np.abs(v).T)
    assert np.all(np.abs(to_np(dh) - ref) <= lim)


@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,k", [(5, 2), (16, 3), (63, 17), (65, 33), (127, 65), (129, 40),
                                 (256, 97), (257, 130), (600, 289), (513, 200)])
def test_int8_products_tile_edges(pk, cplx, n, k):
    """FP64 products on INT8 at the edges of their tiles (256 rows, 32 to 288
    columns), of the 128-byte K chunks and of the 16-byte rows: the bar of the
    FP64 filter (its integer forms of 46 bits or more round less)."""
    announce(f"tile edges: int8 filter n={n} k={k} cplx={cplx}")
    g = np.random.Generator(np.random.PCG64(43 * n + k))
    h, x = _hermitian(g, n, cplx), gen.gaussian(g, (n, k), cplx)
    deg = np.sort(2 * g.integers(1, 5, size=k)).astype(np.int32)
    y_ref, _ = oracle.chebyshev_filter(h, x, deg, 1.05, -1.02, -0.5)
    xt = to_gpu(x)
    with pk.Handle(n, max(1, k - 1), 1, xt.dtype, pk.default_opts(fp64_emulation=14)) as hd:
        y, _ = pk.chase_filter(to_gpu(h), xt, deg, 1.05, -1.02, -0.5, handle=hd)
    y = to_np(y)
    err = np.max(np.abs(y - y_ref), axis=0) / np.max(np.abs(y_ref), axis=0)
    assert err.max() < 1e-12, (int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("prec", ["bf16x3", "bf16x2"])
@pytest.mark.parametrize("cplx", [True, False])
@pytest.mark.parametrize("n,k_wide,ks", [(300, 128, (1, 33, 64, 65, 96, 97)),
                                         (1100, 230, (129, 190, 192, 193)),
                                         (2300, 128, (31, 96)), (3500, 128, (40, 64, 65, 96))])
def test_split_bf16_tiles(pk, cplx, prec, n, k_wide, ks):
    """Split-BF16 products at the tiles their rule picks (64, 128, 192 and 256
    rows by 64, 96 and 128 columns).  Same number of column tiles: the same K
    slices and the same order of every element's sum, so the columns a
    narrower block shares with a wider one are the same bytes.  Against the
    FP64 defect pass: products relative to the residual (1e-4 of the block)
    are off by 2^-16 (three terms) or 2^-8 (two terms), six steps amplify by
    less than 24."""
    announce(f"split-BF16 tiles: {prec} n={n} k={k_wide} {ks} cplx={cplx}")
    code = pk.PREC_BF16X3 if prec == "bf16x3" else pk.PREC_BF16X2
    g = np.random.Generator(np.random.PCG64(47 * n + k_wide))
    z = gen.gaussian(g, (n, n), cplx)
    h = z + z.conj().T
    h = to_gpu(h * (np.sqrt(n) / (2.1 * np.linalg.norm(h))))
    v = np.linalg.qr(gen.gaussian(g, (n, k_wide), cplx))[0]
    r = gen.gaussian(g, (n, k_wide), cplx) * 1e-4 / np.sqrt(n)
    theta = np.linspace(-1.0, -0.6, k_wide)

    def run(k, prec):
        return to_np(pk.chase_filter_ritz(h, to_gpu(v[:, :k].copy()), to_gpu(r[:, :k].copy()),
                                          theta[:k], np.full(k, 6, np.int32), 1.05, -1.02, -0.5,
                                          prec=prec)[0])

    wide, ref = run(k_wide, code), run(k_wide, pk.PREC_FP64)
    tol = 1e-4 * 24 * 2.0 ** (-16 if prec == "bf16x3" else -8)
    assert np.max(np.abs(wide - ref)) <= tol * np.max(np.abs(ref))
    for k in ks:
        assert np.array_equal(run(k, code), wide[:, :k]), k

"""Lanczos coefficients against the oracle on both sides of the block-size
changes of its kernels (256 rows a workgroup, the small-matrix form below
4096 rows, 64-column stages), for every vector count.

Six steps of the three-term recurrence: each coefficient is a sum of at most n
terms of a product with H (error n u ||H||, u = 2^-53, ||H|| = 1 here), and a
step passes earlier errors on with a factor below 1/beta_min, beta about 1/2
on these spectra: 2^6 n u < 4e-11 at n = 5000 bounds it, well below 1e-10."""
import numpy as np
import pytest

import gen
import oracle
from gpu_util import announce, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cplx,n,nvec", [
    (True, 9, 2), (False, 31, 8), (True, 255, 5), (True, 257, 3), (False, 1000, 6), (True, 1025, 4),
    (False, 4095, 7), (False, 4096, 1), (False, 4097, 2)])
def test_lanczos_sizes(cplx, n, nvec):
    import paper_2205_02491_amd as pk
    announce(f"lanczos n={n} nvec={nvec} cplx={cplx}")
    g = np.random.Generator(np.random.PCG64(7 * n + nvec))
    z = gen.gaussian(g, (n, n), cplx)
    h = (z + z.conj().T) / (2.0 * np.sqrt(2.0 * n) if cplx else np.sqrt(8.0 * n))
    s = gen.gaussian(g, (n, nvec), cplx)
    steps = min(6, n)
    runs = oracle.lanczos_runs(h, s, steps)
    with pk.Handle(n, 2, 1, to_gpu(h[:1, :1]).dtype,
                   pk.default_opts(lanczos_vecs=nvec, lanczos_steps=steps)) as hd:
        _, _, _, a, b, lens = pk.chase_lanczos(to_gpu(h), to_gpu(s), handle=hd)
    for r, (ar, br) in enumerate(runs):
        m = min(int(lens[r]), len(ar))
        assert np.max(np.abs(a[r, :m] - ar[:m])) < 1e-10
        assert np.max(np.abs(b[r, :m] - br[:m])) < 1e-10

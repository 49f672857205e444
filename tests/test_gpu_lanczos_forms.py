"""Lanczos coefficients on both sides of the order where the products with H
change from one row a thread to two: 2200 complex, 4096 real (there the sizes
test of the Lanczos step has the real ones).

Tolerance as there: six steps of the recurrence, 2^6 n u < 2e-11 at n = 2201."""
import numpy as np
import pytest

import gen
import oracle
from gpu_util import announce, to_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nvec", [(2199, 4), (2200, 8), (2201, 1), (2201, 3)])
def test_complex_forms(n, nvec):
    import paper_2205_02491_amd as pk
    announce(f"lanczos forms n={n} nvec={nvec}")
    g = np.random.Generator(np.random.PCG64(9 * n + nvec))
    z = gen.gaussian(g, (n, n), True)
    h = (z + z.conj().T) / (2.0 * np.sqrt(2.0 * n))
    s = gen.gaussian(g, (n, nvec), True)
    runs = oracle.lanczos_runs(h, s, 6)
    ht = to_gpu(h)
    with pk.Handle(n, 2, 1, ht.dtype, pk.default_opts(lanczos_vecs=nvec, lanczos_steps=6)) as hd:
        _, _, _, a, b, lens = pk.chase_lanczos(ht, to_gpu(s), handle=hd)
    for r, (ar, br) in enumerate(runs):
        assert int(lens[r]) == len(ar) == 6
        assert np.max(np.abs(a[r] - ar)) < 1e-10
        assert np.max(np.abs(b[r] - br)) < 1e-10

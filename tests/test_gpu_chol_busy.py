"""Cholesky factorisation beside another stream's work: the workgroups of a
panel do not begin together on a busy chip, and all of them have to read the
diagonal block before its factor takes its place.  Every run has the bytes of
the run on an idle chip (each workgroup factors the block in the same order)."""
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cplx", [True, False])
def test_factor_beside_other_work(cplx):
    import torch
    import paper_2205_02491_amd as pk
    dt = torch.complex128 if cplx else torch.float64
    k = 1300
    announce(f"Cholesky beside another stream k={k} cplx={cplx}")
    g = torch.Generator(device="cuda").manual_seed(83 + cplx)
    x = torch.randn(2 * k, k, dtype=dt, device="cuda", generator=g)
    a = torch.matmul(x.mH.contiguous(), x)
    ref, info = pk.chase_cholesky(a)
    assert info == 0
    r = ref.triu()
    err = (torch.matmul(r.mH.contiguous(), r) - a).abs().max() / a.abs().max()
    assert float(err) <= 4 * k * 2.0 ** -53
    m = torch.randn(4096, 4096, dtype=torch.float64, device="cuda", generator=g)
    side, out = torch.cuda.Stream(), torch.empty_like(m)
    torch.cuda.synchronize()
    for _ in range(4):
        with torch.cuda.stream(side):
            for _ in range(3):
                torch.matmul(m, m, out=out)
        got, info = pk.chase_cholesky(a)
        assert info == 0 and torch.equal(got, ref)
    torch.cuda.synchronize()

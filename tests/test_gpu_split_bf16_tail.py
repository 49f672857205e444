"""Split-BF16 products where the split-K tail begins inside a row of tiles.

More than 256 tiles of 256 x 128 run in rounds of 256; the last, nearly empty
round is cut along K.  With three column tiles its first tile may be the second
or third of its row (n = 21800: 86 x 3 tiles, the last two cut).  Whether an
element's sum is cut must depend on that plan alone and not on how wide the
column tiles are made, or a block of 260 columns (96 wide) and one of 300 (128
wide), equal in the columns they share, end in different bytes there."""
import numpy as np
import pytest

from gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["bf16x3", "bf16x2"])
@pytest.mark.parametrize("cplx", [True, False])
def test_tail_inside_a_tile_row(cplx, prec):
    import torch
    import paper_2205_02491_amd as pk
    n, wide, narrow = 21800, 300, 260
    announce(f"split-BF16 tail inside a tile row: {prec} cplx={cplx}")
    code = pk.PREC_BF16X3 if prec == "bf16x3" else pk.PREC_BF16X2
    dt = torch.complex128 if cplx else torch.float64
    g = torch.Generator(device="cuda").manual_seed(61 + cplx)
    h = torch.randn(n, n, dtype=dt, device="cuda", generator=g)
    h = h.add(h.mH).div_(2.0 * (2.0 * n) ** 0.5)
    v = torch.randn(n, wide, dtype=dt, device="cuda", generator=g) / n ** 0.5
    r = torch.randn(n, wide, dtype=dt, device="cuda", generator=g) * (1e-4 / n ** 0.5)
    theta = np.linspace(-1.0, -0.6, wide)

    def run(k):
        return pk.chase_filter_ritz(h, v[:, :k].contiguous(), r[:, :k].contiguous(), theta[:k],
                                    np.full(k, 4, np.int32), 1.05, -1.02, -0.5, prec=code)[0]

    a, b = run(narrow), run(wide)[:, :narrow]
    bad = (a != b).nonzero()
    assert bad.numel() == 0, (bad.shape[0], bad[0].tolist(), bad[-1].tolist())

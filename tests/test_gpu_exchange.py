"""Exchanges of the strided passes at the lengths with a factor 9, whose stages
fill blocks of 6, 12 or 18 positions, whose middle radix is not a multiple of
the last one (288 = 12 6 4) or has more butterflies per thread than one (576 =
12 12 4), and whose butterflies per thread are odd in number: every form of the
exchange gives the bits of the whole-buffer one, in both tiers."""
import pytest

from paper_2506_04489_amd import psp as B
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [54, 108, 144, 162, 216, 288, 324])
def test_every_exchange_gives_the_same_bits(n, dtype):
    import torch
    announce("exchange n=%d %s" % (n, dtype))
    g = torch.Generator().manual_seed(n)
    rho = torch.randn((n,) * 3, generator=g, dtype=torch.float64)
    rho = rho.to(torch.float64 if dtype == "f64" else torch.float32).cuda()
    p = B.Plan(n, 2.0 / n, 40, dtype=dtype).precompute().set_shape([0] * 5, [0] * 5)
    p.profile_enable(19)                    # five passes at every length
    want = p.solve(rho)
    for tile in range(1, 7):
        for q in (1, 2, 3):
            p.set_shape([0] * 5, [tile if i == q else 0 for i in range(5)])
            u = p.solve(rho)
            torch.cuda.synchronize()
            assert torch.equal(u, want), (tile, q)
    p.close()

"""Exchanges of the strided passes whose last (inverse: first) two stages stay
inside a wave, at the lengths whose middle radix is not a multiple of the last
one (288 = 12 6 4) or has more butterflies per thread than one (576 = 12 12 4):
every form of the exchange gives the bits of the whole-buffer one."""
import pytest

from paper_2506_04489_amd import psp as B
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [144, 288])
def test_every_exchange_gives_the_same_bits(n):
    import torch
    announce("exchange n=%d" % n)
    g = torch.Generator().manual_seed(n)
    rho = torch.randn((n,) * 3, generator=g, dtype=torch.float64).cuda()
    p = B.Plan(n, 2.0 / n, 40).precompute().set_shape([0] * 5, [0] * 5)
    want = p.solve(rho)
    for tile in range(1, 7):
        for q in (1, 2, 3):
            p.set_shape([0] * 5, [tile if i == q else 0 for i in range(5)])
            u = p.solve(rho)
            torch.cuda.synchronize()
            assert torch.equal(u, want), (tile, q)
    p.close()

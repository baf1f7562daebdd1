"""Replays of a recorded single solve (made as kernel launches) on streams of
their own: ordered after the stream's earlier work, bitwise psp_solve, for a
solve of one launch, of three and of five, and for a grid."""
import pytest

from paper_2506_04489_amd import psp as B
from tests.gpu_util import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 48, 96, (16, 24, 36)])
def test_replays_follow_their_stream(n):
    import torch
    announce("replay %s" % (n,))
    ns = n if isinstance(n, tuple) else (n,) * 3
    p = B.Plan(n, 0.05 if not isinstance(n, tuple) else (0.05,) * 3, 40).precompute()
    g = torch.Generator().manual_seed(3)
    base = torch.randn(ns, generator=g, dtype=torch.float64).cuda()
    rho, u = base.clone(), torch.empty_like(base)
    rec = B.Graph.capture(p, rho, u)
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    outs = []
    with torch.cuda.stream(st):
        for k in range(3):
            rho.copy_(base * (k + 1))            # ordered before the replay on st
            rec.launch()
            outs.append(u.clone())
    st.synchronize()
    for k, o in enumerate(outs):
        want = p.solve(base * (k + 1))
        torch.cuda.synchronize()
        assert torch.equal(o, want), k
    rec.close()

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


@pytest.mark.parametrize("n", [48, 96, 108])
def test_threads_replay_one_record_on_one_stream(n):
    """Replays of one record by several threads on one stream follow one another
    whole: their launches share a workspace that the passes update in place."""
    import threading

    import torch
    announce("replay by threads %d" % n)
    g = torch.Generator().manual_seed(5)
    rho = torch.randn((n,) * 3, generator=g, dtype=torch.float64).cuda()
    p = B.Plan(n, 2.0 / n, 40).precompute()
    want = p.solve(rho)
    u = torch.empty_like(rho)
    rec = B.Graph.capture(p, rho, u)
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(20):
        u.zero_()
        torch.cuda.synchronize()
        go, errors = threading.Barrier(4), []

        def replay():
            try:
                go.wait(timeout=30)
                for _ in range(8):
                    rec.launch(stream=st)
            except Exception as e:          # reported below, in the test's thread
                errors.append(e)

        threads = [threading.Thread(target=replay) for _ in range(4)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        st.synchronize()
        assert not errors
        assert torch.equal(u, want)
    rec.close()

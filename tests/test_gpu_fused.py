"""The three-launch solve of cubes with n <= 72, 96 and 128 (fused.hpp): bitwise equal to
the five passes at every length it is built for, in both tiers, on inputs of
full power.  Five passes run when the solve records per-pass events, when k3
runs in chunks, or when a radix plan differs from the fused one."""
import pytest

from oracle import psp_oracle as O
from paper_2506_04489_amd import psp as B
from tests.gpu_util import announce, rel_max_err

pytestmark = pytest.mark.gpu

FUSED = [4, 6, 8, 12, 16, 18, 24, 32, 36, 48, 54, 64, 72, 96, 128]


@pytest.fixture(autouse=True)
def _name(request):
    announce(request.node.nodeid)
    yield


def _noise(n, dtype, seed):
    import torch
    g = torch.Generator().manual_seed(seed)
    v = torch.randn((n,) * 3, generator=g, dtype=torch.float64)
    return v.to(torch.float64 if dtype == "f64" else torch.float32).cuda()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", FUSED)
def test_fused_equals_the_five_passes_bitwise(n, dtype):
    import torch
    rho = _noise(n, dtype, 50 + n)
    B.debug_guards(True)
    try:
        p = B.Plan(n, 2.0 / n, 40, dtype=dtype).precompute()
        u = p.solve(rho)
        p.profile_enable(1)
        five = p.solve(rho)
        torch.cuda.synchronize()
        assert p.profile_read()[0] == 1
        assert torch.equal(u, five)
        assert p.guards_intact()
        p.set_tuning(1, 0)                       # chunks of one k3 tile: five passes
        chunked = p.solve(rho)
        torch.cuda.synchronize()
        assert torch.equal(u, chunked)
        p.set_tuning(0, 0)
        # several solves in one launch, and without an allocation
        rhos = [_noise(n, dtype, 500 + i) for i in range(3)]
        us = [torch.empty_like(r) for r in rhos]
        B.solve_batched([p] * 3, rhos, us)
        v = torch.empty_like(rho)
        for r, w in zip(rhos, us):
            p.solve_noalloc(r, v)
            torch.cuda.synchronize()
            assert torch.equal(v, w)
        p.close()
    finally:
        B.debug_guards(False)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", FUSED)
def test_batched_fused_solves_stay_inside_their_workspaces(n, dtype):
    """The tiles that several solves per launch take, in guarded workspaces: a
    stream of its own has a pool of its own, allocated by this batch."""
    import ctypes

    import torch
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))
    st = ctypes.c_void_p()
    rhos = [_noise(n, dtype, 900 + i) for i in range(3)]
    us = [torch.empty_like(r) for r in rhos]
    p = B.Plan(n, 2.0 / n, 40, dtype=dtype).precompute()
    torch.cuda.synchronize()
    assert hip.hipStreamCreate(ctypes.byref(st)) == 0
    B.debug_guards(True)
    try:
        B.solve_batched([p] * 3, rhos, us, stream=st.value)
        torch.cuda.synchronize()
        assert p.guards_intact()
    finally:
        B.debug_guards(False)
    for r, u in zip(rhos, us):
        want = p.solve(r)
        torch.cuda.synchronize()
        assert torch.equal(u, want)
    p.close()

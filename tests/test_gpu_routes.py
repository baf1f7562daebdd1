"""How many kernels a cube's solve launches: one or three where its plan starts
from the tuning table, the five passes where a shape was set, so that a sweep of
tiles runs the tiles it names.  Counted as the kernel nodes of a captured solve."""
import ctypes

import pytest

from paper_2506_04489_amd import psp as B
from tests.gpu_util import TILES, announce

pytestmark = pytest.mark.gpu


def _hip():
    import torch  # noqa: F401  (loads the HIP runtime)
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    return ctypes.CDLL(path)


def launches(plan, rho):
    """Kernel nodes of one captured solve of `plan` (nothing is executed)."""
    return len(block_sizes(plan, rho))


def block_sizes(plan, rho):
    """Threads per workgroup of the kernels of a captured solve, in order."""
    import torch
    hip, st = _hip(), torch.cuda.Stream()
    u = torch.empty_like(rho)
    s, graph, count = ctypes.c_void_p(st.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t()
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(s, 2) == 0          # relaxed
    try:
        plan.solve_noalloc(rho, u, stream=st)
    finally:
        rc = hip.hipStreamEndCapture(s, ctypes.byref(graph))
    assert rc == 0 and hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(count)) == 0
    sizes = []
    for node in nodes:
        kind, params = ctypes.c_int(-1), (ctypes.c_uint32 * 64)()       # blockDim comes first
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0 and kind.value == 0
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), params) == 0
        sizes.append(params[0])
    assert hip.hipGraphDestroy(graph) == 0
    return sizes


def _noise(n, dtype):
    import torch
    g = torch.Generator().manual_seed(n)
    v = torch.randn((n,) * 3, generator=g, dtype=torch.float64)
    return v.to(torch.float64 if dtype == "f64" else torch.float32).cuda()


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [4, 8, 16, 18, 24, 36, 48, 64, 128])
def test_a_set_shape_runs_its_five_passes(n, dtype):
    import torch
    announce("routes n=%d %s" % (n, dtype))
    rho = _noise(n, dtype)
    p = B.Plan(n, 2.0 / n, 40, dtype=dtype).precompute()
    assert launches(p, rho) == (1 if n <= 8 else 3)
    u = p.solve(rho)
    plan, _ = p.shape()
    for r in (0, 1, 5, 20):
        p.set_shape(plan, [r % c for c in TILES])
        assert launches(p, rho) == 5
        v = p.solve(rho)
        torch.cuda.synchronize()
        assert torch.equal(u, v), r
    p.close()


@pytest.mark.parametrize("n,dtype", [(8, "f64"), (48, "f64"), (64, "f32"), (72, "f64"), (96, "f32")])
def test_the_autotuned_route_is_the_one_solves_take(n, dtype):
    import torch
    announce("autotuned route n=%d %s" % (n, dtype))
    old = B.tuning_get(n, dtype)
    rho = _noise(n, dtype)
    try:
        p = B.Plan(n, 2.0 / n, 40, dtype=dtype).precompute()
        p.autotune(reps=1)
        count = launches(p, rho)
        # one solve of these lengths takes five passes whatever the plans
        assert count == 5 if n in (72, 96) else count in (1, 3, 5)
        q = B.Plan(n, 2.0 / n, 40, dtype=dtype).precompute()    # from the table
        assert q.shape() == p.shape() and launches(q, rho) == count
        u = p.solve(rho)
        p.profile_enable(1)                                     # five passes
        five = p.solve(rho)
        torch.cuda.synchronize()
        assert torch.equal(u, five)
    finally:
        B.tuning_set(n, dtype, *old)


@pytest.mark.parametrize("ns,dtype,few", [((192, 8, 48), "f64", True), ((192, 54, 36), "f64", True),
                                          ((192, 128, 48), "f64", False), ((256, 8, 48), "f32", True),
                                          ((256, 96, 96), "f32", False)])
def test_a_grids_i1_pass_has_all_threads_where_columns_are_few(ns, dtype, few):
    import torch
    announce("i1 pass of %s %s" % (ns, dtype))
    n, (plan, tile) = ns[0], B.tuning_get(ns[0], dtype)
    g = torch.Generator().manual_seed(1)
    rho = torch.randn(ns, generator=g, dtype=torch.float64).cuda()
    rho = rho.to(torch.float64 if dtype == "f64" else torch.float32)
    sizes, us = {}, {}
    try:
        for t in (2, 4):                # half-size exchanges, all threads and half of them
            B.tuning_set(n, dtype, plan, [t if q == 2 else x for q, x in enumerate(tile)])
            p = B.Plan(ns, tuple(2.0 / m for m in ns), 40, dtype=dtype).precompute()
            sizes[t], us[t] = block_sizes(p, rho), p.solve(rho)
            torch.cuda.synchronize()
            p.close()
    finally:
        B.tuning_set(n, dtype, plan, tile)
    assert (sizes[2] == sizes[4]) == few, sizes
    assert torch.equal(us[2], us[4])

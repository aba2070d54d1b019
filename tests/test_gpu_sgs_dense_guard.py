"""When the dense form up to 8192 tokens keeps the incremental greedy's result and
when its float64 sweeps write it: the outputs tell, bit for bit, as the
gains and objectives of the two are sums on a fixed grid and in float64.  The
sweeps alone run in a workspace of their own size."""
import ctypes

import numpy as np
import pytest

from tests.test_gpu_sgs_dense_route import _sweep_bytes
from tests.test_gpu_sgs_order import group_width, scene

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cost(n, seed, low=0.0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    cost = low + (3.0 - low) * torch.rand(n, n, device="cuda", generator=g)
    cost.fill_diagonal_(0.0)
    return cost, torch.rand(n, device="cuda", generator=g)


def _sweeps(cost, cap, k, c0):
    import paper_2608_13226_amd as cp
    small = torch.empty(_sweep_bytes(cost.shape[0], k), dtype=torch.uint8, device="cuda")
    return cp.sgs_select(cost, cap, k, c0=c0, check=True, workspace=small)


def _equal(a, b):
    return all(torch.equal(x, y) for x, y in ((a.selected, b.selected), (a.gain, b.gain),
                                              (a.objective, b.objective), (a.assign, b.assign)))


# Few picks do not pay for the incremental form: the line depends on n.
@pytest.mark.parametrize("n,last", [(1000, 12), (1001, 7), (2049, 7), (3000, 19), (4096, 22), (6000, 16), (8192, 10)])
def test_few_picks_take_the_sweeps_alone(n, last):
    import paper_2608_13226_amd as cp
    cost, cap = _cost(n, n)
    for k in (last, last + 1):
        print(f"sgs dense guard few picks n={n} k={k}", flush=True)
        full, ref = cp.sgs_select(cost, cap, k, c0=3.0, check=True), _sweeps(cost, cap, k, 3.0)
        assert torch.equal(full.selected, ref.selected)
        assert _equal(full, ref) == (k == last)


# 2500 tokens and more: the early kernel, whose launches the check also covers.
@pytest.mark.parametrize("n,k", [(300, 40), (2049, 21), (2500, 60), (8192, 40)])
def test_ordinary_data_keep_the_incremental_result(n, k):
    import paper_2608_13226_amd as cp
    cost, cap = _cost(n, n)
    print(f"sgs dense guard ordinary n={n}", flush=True)
    full = cp.sgs_select(cost, cap, k, c0=3.0, check=True)
    inc = cp.sgs_select(cost, cap, k, c0=3.0, incremental=True, check=True)
    assert _equal(full, inc)
    assert not _equal(full, _sweeps(cost, cap, k, 3.0))


@pytest.mark.parametrize("n,k", [(300, 40), (2500, 60), (8192, 40)])
@pytest.mark.parametrize("what", ["cost", "cost nan", "capacity", "capacity inf"])
def test_one_entry_outside_the_domain(n, k, what):
    import paper_2608_13226_amd as cp
    cost, cap = _cost(n, n + 1)
    if what == "cost":
        cost[n - 1, n - 2] = -0.25
    elif what == "cost nan":
        cost[n - 1, n - 1] = float("nan")
    else:
        cap[n - 1] = -1e-3 if what == "capacity" else float("inf")
    print(f"sgs dense guard {what} n={n}", flush=True)
    full = cp.sgs_select(cost, cap, k, c0=3.0, check=True)
    ref = _sweeps(cost, cap, k, 3.0)
    for x, y in ((full.selected, ref.selected), (full.gain, ref.gain), (full.objective, ref.objective),
                 (full.assign, ref.assign)):
        assert torch.equal(x.nan_to_num(nan=-7.0) if x.is_floating_point() else x,
                           y.nan_to_num(nan=-7.0) if y.is_floating_point() else y)


def test_beyond_the_bound_the_workspace_is_the_sweeps():
    import paper_2608_13226_amd as cp
    n, k = 8193, 12
    lib = cp.library()
    assert lib.coverprune_sgs_workspace(n, k, cp.CP_SGS_DENSE) == _sweep_bytes(n, k)
    cost, cap = _cost(n, 3)
    print("sgs dense guard n=8193", flush=True)
    assert _equal(cp.sgs_select(cost, cap, k, c0=3.0, check=True), _sweeps(cost, cap, k, 3.0))


# The grid follows c0: far above the costs it does not resolve their
# differences, and float64 does.
@pytest.mark.parametrize("c0", [1e7, 1e9, 1e15])
@pytest.mark.parametrize("n,k", [(1024, 30), (2500, 40)])
def test_uncovered_cost_far_above_the_costs(n, k, c0):
    import paper_2608_13226_amd as cp
    cost, cap = _cost(n, 5)
    print(f"sgs dense guard c0={c0} n={n}", flush=True)
    assert _equal(cp.sgs_select(cost, cap, k, c0=c0, check=True), _sweeps(cost, cap, k, c0))


def test_late_gains_from_small_capacities():
    # The large capacities are all covered after a few picks; the others lie
    # 2^-25 below them.
    import paper_2608_13226_amd as cp
    n, k = 1024, 60
    cost, cap = _cost(n, 6, low=2.5)
    cap = (cap + 0.5) * 2.0 ** -25
    cap[:16] = 1.0
    cost[:16] = 0.0
    print("sgs dense guard small capacities", flush=True)
    assert _equal(cp.sgs_select(cost, cap, k, c0=3.0, check=True), _sweeps(cost, cap, k, 3.0))


def test_all_targets_covered():
    import paper_2608_13226_amd as cp
    n, k = 600, 90
    g = torch.Generator(device="cuda").manual_seed(8)
    at = torch.randint(0, 50, (n,), device="cuda", generator=g)
    small, cap = _cost(50, 9)
    cost = small[at][:, at].contiguous()
    cap = torch.rand(n, device="cuda", generator=g)
    print("sgs dense guard covered", flush=True)
    full, ref = cp.sgs_select(cost, cap, k, c0=3.0, check=True), _sweeps(cost, cap, k, 3.0)
    assert float(ref.objective[-1]) == 0.0
    assert _equal(full, ref)


# Pairs of candidates whose gains differ by 2^-38: the sweeps compare exactly
# within strips of 256 columns, the incremental form within groups of 64.
@pytest.mark.parametrize("n,pairs,idle,early,long", [(300, 30, 0, 0, 0), (2400, 60, 560, 9, 8)])
def test_near_ties_are_the_sweeps(n, pairs, idle, early, long):
    import paper_2608_13226_amd as cp
    c, v, want = scene(n, pairs, idle, early, long, group_width(n), n)
    cost, cap = torch.from_numpy(np.ascontiguousarray(c.T)).cuda(), torch.from_numpy(v).cuda()
    print(f"sgs dense guard near ties n={n}", flush=True)
    ref = _sweeps(cost, cap, pairs, 3.0)
    assert ref.selected.tolist() != want
    assert _equal(cp.sgs_select(cost, cap, pairs, c0=3.0, check=True), ref)


def test_without_gains_and_objectives():
    import paper_2608_13226_amd as cp
    n, k = 500, 30
    lib = cp.library()
    cost, cap = _cost(n, 11)
    for c0 in (3.0, 1e9):
        print(f"sgs dense guard picks only c0={c0}", flush=True)
        sel = torch.empty(k, dtype=torch.int32, device="cuda")
        ws = torch.empty(lib.coverprune_sgs_workspace(n, k, cp.CP_SGS_DENSE), dtype=torch.uint8, device="cuda")
        p = lambda t: ctypes.c_void_p(t.data_ptr())
        st = lib.coverprune_sgs_select(p(cost), n, p(cap), k, c0, cp.CP_SGS_DENSE, p(sel), None, None, None, p(ws),
                                       ws.numel(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0
        torch.cuda.synchronize()
        assert torch.equal(sel, _sweeps(cost, cap, k, c0).selected)


@pytest.mark.parametrize("n,k", [(600, 100), (3000, 120)])
def test_smooth_gains(n, k):
    # Neighbours on a line have nearly equal gains: whether a pick among them
    # is the sweeps' is seen, so the result is theirs either way.
    import paper_2608_13226_amd as cp
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.rand(n, 1, device="cuda", generator=g)
    cost = (3.0 * (x - x.t()).abs()).contiguous()
    cap = torch.full((n,), 1.0 / n, device="cuda")
    print(f"sgs dense guard line n={n}", flush=True)
    full, ref = cp.sgs_select(cost, cap, k, c0=3.0, check=True), _sweeps(cost, cap, k, 3.0)
    assert torch.equal(full.selected, ref.selected) and torch.equal(full.assign, ref.assign)
    assert torch.allclose(full.gain, ref.gain, rtol=2.0 ** -30, atol=0.0)
    assert torch.allclose(full.objective, ref.objective, rtol=2.0 ** -36, atol=0.0)

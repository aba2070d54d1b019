"""The rows schedule's list phase (rounds of picks among the best candidates)
against the compact schedule, which has none: the same integers, so the same
outputs bit for bit.  Costs are made so that each way through a round is
taken: lists that hold every pair, candidates with more pairs than a list
holds, blocks whose own pairs do not fit in LDS, exact ties and zero gains."""
import numpy as np
import pytest

from oracle import sgs
from tests import parity

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _cost(kind, n, rng):
    if kind == "falling":
        # A candidate's cost to every other target falls with its index: the
        # candidates above the last pick keep a pair with nearly all targets.
        c = np.repeat((1.0 - 1e-3 * np.arange(n) / n)[:, None], n, axis=1) + 1e-5 * rng.random((n, n))
    elif kind == "random":
        c = 3.0 * rng.random((n, n))
    elif kind == "ties":
        # Few distinct costs, duplicated candidates: many equal gains.
        c = rng.integers(1, 6, (n, n)) * 0.5
        c[1::7] = c[0::7][:len(c[1::7])]
    else:                                       # "clusters": tight groups, gains that reach 0
        p = rng.integers(0, max(2, n // 40), n).astype(np.float64)[:, None] + 0.02 * rng.random((n, 2))
        c = np.minimum(np.abs(p[:, None, 0] - p[None, :, 0]) + np.abs(p[:, None, 1] - p[None, :, 1]), 3.0)
        c[np.abs(c) < 0.01] = 0.0
    c = c.astype(np.float32)
    np.fill_diagonal(c, 0.0)
    return c                                    # source-major


# Edges: one block and several, W that no power of two divides, budgets just
# past the first list step (8 steps, n / 128 from 1024 tokens on), lists in
# place of the rows of T (k <= 128) and of their own, capacities in LDS
# (n <= 8192) and not.
CASES = [("clusters", 33, 33), ("ties", 137, 40), ("random", 256, 30), ("random", 257, 200), ("falling", 1000, 100),
         ("ties", 1023, 150), ("random", 1025, 129), ("clusters", 1040, 600), ("falling", 2500, 60),
         ("random", 4097, 140), ("clusters", 8192, 300), ("clusters", 8193, 300)]


@pytest.mark.parametrize("kind,n,k", CASES)
def test_rounds_equal_the_compact_schedule(kind, n, k):
    import paper_2608_13226_amd as cp
    print(f"sgs lists {kind} n={n} k={k}", flush=True)
    rng = np.random.default_rng(n)
    c = _cost(kind, n, rng)
    v = rng.random(n).astype(np.float32)
    if kind == "ties":
        v[:] = 1.0
    v /= v.sum()
    cost = torch.from_numpy(c).cuda().t().contiguous()
    cap = torch.from_numpy(v).cuda()
    rows = cp.sgs_select(cost, cap, k, c0=3.0, incremental=True, check=True)
    compact = cp.sgs_select(cost, cap, k, c0=3.0, incremental=True, compact=True, check=True)
    for x, y in zip((rows.selected, rows.gain, rows.objective, rows.assign),
                    (compact.selected, compact.gain, compact.objective, compact.assign)):
        assert torch.equal(x, y)
    if n <= 1100:
        ties, g_or, o_or = parity.replay_greedy(c, v, 3.0, rows.selected.cpu().numpy())
        assert np.allclose(rows.gain.cpu().numpy(), g_or, rtol=1e-6, atol=1e-12)
        assert np.allclose(rows.objective.cpu().numpy(), o_or, rtol=1e-9, atol=1e-12)
        if not ties:
            ref = sgs.sgs_ref(c.astype(np.float64), v.astype(np.float64), k, 3.0)
            assert np.array_equal(rows.selected.cpu().numpy(), ref["selected"])


def test_rounds_in_a_batch_with_wide_blocks():
    # Four scenes of 6000 tokens: 64 blocks each, 94 columns a block (two per
    # lane), and one small scene without a list phase.
    import paper_2608_13226_amd as cp
    print("sgs lists batch", flush=True)
    sizes, ks = [6000, 6000, 6000, 5999, 40], [130, 90, 60, 200, 10]
    costs, caps = [], []
    for i, n in enumerate(sizes):
        rng = np.random.default_rng(50 + i)
        c = _cost("clusters" if i != 2 else "random", n, rng)
        v = rng.random(n).astype(np.float32)
        costs.append(torch.from_numpy(c).cuda().t().contiguous())
        caps.append(torch.from_numpy(v / v.sum()).cuda())
    got = cp.sgs_select_batch(costs, caps, ks, c0=3.0, check=True)
    for c, v, k, r in zip(costs, caps, ks, got):
        one = cp.sgs_select(c, v, k, c0=3.0, incremental=True, compact=True, check=True)
        for x, y in zip((r.selected, r.gain, r.objective, r.assign), (one.selected, one.gain, one.objective, one.assign)):
            assert torch.equal(x, y)


# Picks past the last gain, four a round: targets without capacity still change
# hands, in the order of the picks.
@pytest.mark.parametrize("kind", ["constant", "few targets", "few groups"])
@pytest.mark.parametrize("n,k", [(300, 129), (300, 300), (1001, 500), (2500, 250), (5070, 700)])
def test_picks_of_no_gain(n, k, kind):
    import paper_2608_13226_amd as cp
    rng = np.random.default_rng(n + k)
    v = rng.random(n).astype(np.float32)
    if kind == "constant":
        c = np.full((n, n), 1.5, np.float32)
    elif kind == "few targets":
        c = (3.0 * rng.random((n, n))).astype(np.float32)
        v[rng.permutation(n)[40:]] = 0.0
    else:
        at = rng.integers(0, 30, n)
        c = (3.0 * rng.random((30, 30))).astype(np.float32)[at][:, at]
    if kind != "constant":
        np.fill_diagonal(c, 0.0)
    cost, cap = torch.from_numpy(c).cuda().t().contiguous(), torch.from_numpy(v / v.sum()).cuda()
    print(f"sgs lists no gain {kind} n={n} k={k}", flush=True)
    one = cp.sgs_select(cost, cap, k, c0=3.0, incremental=True, compact=True, check=True)
    assert kind == "few groups" or float(one.gain[-1]) == 0.0
    r = cp.sgs_select(cost, cap, k, c0=3.0, incremental=True, check=True)
    for x, y in zip((r.selected, r.gain, r.objective, r.assign), (one.selected, one.gain, one.objective, one.assign)):
        assert torch.equal(x, y)

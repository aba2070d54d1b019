"""The rows kernel between the early kernel and the list phase with no, one, two
or three steps of its own (2304 tokens: the lists take over at step 18), alone
and in a batch.  With one step, or two of which the second is predicted, it
ends without waiting for another block, so what it hands over must not lie
where a late block still reads what it resumes from.  Against the
compact schedule, which hands nothing over: the same outputs bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N, K, FIRST = 2304, 90, 18


def _scene(dense_steps, seed):
    """Picks 0 .. K - 1 are known: token i of them covers itself, for falling
    weights.  The first `dense_steps` also lower 600 targets of no
    weight each; the step after them lowers one target only, which ends
    the early kernel."""
    rng = np.random.default_rng(seed)
    order = rng.permutation(N)
    picks, idle, rest = order[:K], order[K:K + 600], order[K + 600:]
    c = np.full((N, N), 3.0, np.float32)                    # source-major
    c[np.ix_(rest, rest)] = 2.0 + rng.random((len(rest), len(rest)))
    for i, p in enumerate(picks):
        c[p, idle] = 2.9 - 0.01 * i if i < dense_steps else 2.95
    np.fill_diagonal(c, 0.0)
    v = np.zeros(N, np.float32)
    v[picks] = 1.0 - np.arange(K) / 1000.0
    v[rest] = 1e-5 * rng.random(len(rest))
    return torch.from_numpy(np.ascontiguousarray(c.T)).cuda(), torch.from_numpy(v).cuda(), picks


def _same(r, one):
    for x, y in zip((r.selected, r.gain, r.objective, r.assign), (one.selected, one.gain, one.objective, one.assign)):
        assert torch.equal(x, y)


# The early kernel ends after the step that follows the dense ones.
@pytest.mark.parametrize("own_steps", [0, 1, 2, 3])
def test_few_steps_between_the_early_kernel_and_the_lists(own_steps):
    import paper_2608_13226_amd as cp
    scenes = [_scene(FIRST - 1 - own_steps, 7 + own_steps + 10 * i) for i in range(2)]
    compact = []
    for i, (cost, cap, picks) in enumerate(scenes):
        print(f"sgs handover own_steps={own_steps} scene {i}", flush=True)
        one = cp.sgs_select(cost, cap, K, c0=3.0, incremental=True, compact=True, check=True)
        assert one.selected.tolist() == picks.tolist()
        _same(cp.sgs_select(cost, cap, K, c0=3.0, incremental=True, check=True), one)
        compact.append(one)
    print(f"sgs handover own_steps={own_steps} batch", flush=True)
    got = cp.sgs_select_batch([s[0] for s in scenes], [s[1] for s in scenes], [K, K], c0=3.0, check=True)
    for r, one in zip(got, compact):
        _same(r, one)

"""Which of two candidates with nearly equal gains is picked.  Candidates of one
group of ceil(n / ceil(n / 64)) consecutive tokens compare by their exact gains,
others to 2^-31 relative, then by index, in every form of the incremental
greedy and in every phase of it.

A scene holds pairs of candidates a < b over targets of their own, with
gain(b) = gain(a) (1 + 2^-38): b comes first inside a group, a across groups.
The weights of the pairs fall, so the picks are known.  All values are small
multiples of powers of two: every sum is exact."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def group_width(n, per=64):
    return -(-n // -(-n // per))


def scene(n, pairs, idle, early, long, width, seed):
    """`idle` targets of no weight are lowered by each of the first `early` pairs (steps with many hits), another
    `idle` by the last `long` pairs (candidates with more targets than a list holds)."""
    rng = np.random.default_rng(seed)
    free = np.ones(n, bool)
    ab = []
    for i in range(pairs):
        # Close together (one block), one group apart at most, anywhere: in turn.
        while True:
            a = int(rng.integers(0, n - 1))
            b = int(min(n - 1, a + 1 + rng.integers(0, (6, width, n)[i % 3])))
            if a < b and free[a] and free[b]:
                break
        free[[a, b]] = False
        ab.append((a, b))
    rest = rng.permutation(np.nonzero(free)[0])
    j1, j2, z1, z2 = np.split(rest[:2 * pairs + 2 * idle], [pairs, 2 * pairs, 2 * pairs + idle])
    c = np.full((n, n), 3.0, np.float32)                    # source-major
    v = np.zeros(n, np.float32)
    for i, (a, b) in enumerate(ab):
        v[j1[i]] = 1.0 - i * 2.0 ** -8
        v[j2[i]] = v[j1[i]] * 2.0 ** -20
        c[[a, b], j1[i]] = 2.0
        c[b, j2[i]] = 3.0 - 2.0 ** -18
        if idle and i < early:
            c[np.ix_([a, b], z1)] = 2.9 - 0.01 * i
        if idle and i >= pairs - long:
            c[np.ix_([a, b], z2)] = 2.9 - 0.01 * i
    same = [a // width == b // width for a, b in ab]
    assert any(same) and not all(same)
    return c, v, [b if x else a for x, (a, b) in zip(same, ab)]


def _cuda(c, v):
    return torch.from_numpy(np.ascontiguousarray(c.T)).cuda(), torch.from_numpy(v).cuda()


# 300 tokens: rows and list kernels; 2400 and 5070: early, rows and list, blocks of 16 and 20 columns, groups of 64.
SCENES = [(300, 30, 0, 0, 0), (2400, 60, 560, 9, 8), (5070, 100, 560, 30, 0)]


@pytest.mark.parametrize("n,pairs,idle,early,long", SCENES)
def test_near_ties_inside_and_across_groups(n, pairs, idle, early, long):
    import paper_2608_13226_amd as cp
    width = group_width(n)
    c, v, want = scene(n, pairs, idle, early, long, width, n)
    cost, cap = _cuda(c, v)
    for name, kw in (("rows", {}), ("compact", dict(compact=True))):
        print(f"sgs order {name} n={n}", flush=True)
        r = cp.sgs_select(cost, cap, pairs, c0=3.0, incremental=True, check=True, **kw)
        assert r.selected.tolist() == want, name
    print(f"sgs order batch n={n}", flush=True)
    for r in cp.sgs_select_batch([cost, cost], [cap, cap], [pairs, pairs], c0=3.0, check=True):
        assert r.selected.tolist() == want


# Without and with chains of predicted winners.
@pytest.mark.parametrize("pairs", [60, 120])
def test_near_ties_in_the_local_greedy(pairs):
    import paper_2608_13226_amd as cp
    n = 2400
    c, v, want = scene(n, pairs, 0, 0, 0, group_width(n), 3)
    nbr = np.repeat(np.arange(n)[:, None], 4, axis=1)       # cost 3.0 to oneself: no gain
    for i in range(n):
        j = np.nonzero(c[i] < 3.0)[0]
        nbr[i, :len(j)] = j
    cost, cap = _cuda(c, v)
    print("sgs order local", flush=True)
    r = cp.sgs_local_select(cost, cap, torch.from_numpy(nbr.astype(np.int32)).cuda(), pairs, c0=3.0, check=True)
    assert r.selected.tolist() == want


def batch_widths(sizes, units=256):
    """Tokens per group of each scene of a batch: every scene has one block, then the one with the most tokens
    a block gains one (up to one per 64 tokens) until the compute units run out."""
    nb = [1] * len(sizes)
    for _ in range(units - len(sizes)):
        wide = [-(-n // b) if b < -(-n // 64) else 0 for n, b in zip(sizes, nb)]
        if max(wide) == 0:
            break
        nb[wide.index(max(wide))] += 1
    return [-(-n // b) for n, b in zip(sizes, nb)]


def test_near_ties_of_a_small_scene_beside_large_ones():
    # The large scenes get blocks of more than 64 columns, and one kernel serves
    # all of the batch: the small one's groups hold there too.
    import paper_2608_13226_amd as cp
    n, pairs = 300, 30
    width = batch_widths([6000] * 4 + [n])[-1]
    assert width > 64
    c, v, want = scene(n, pairs, 0, 0, 0, width, 300)
    cost, cap = _cuda(c, v)
    g = torch.Generator(device="cuda").manual_seed(4)
    big = [3.0 * torch.rand(6000, 6000, device="cuda", generator=g) for _ in range(4)]
    caps = [torch.rand(6000, device="cuda", generator=g) for _ in range(4)]
    for k in (20, 100):                                     # without and with the list kernel
        print(f"sgs order mixed batch k={k}", flush=True)
        r = cp.sgs_select_batch(big + [cost], caps + [cap], [k] * 4 + [pairs], c0=3.0, check=True)
        assert r[-1].selected.tolist() == want

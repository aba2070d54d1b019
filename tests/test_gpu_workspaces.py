"""Workspaces smaller than the ones the library asks for, which calls with an
older and slower way still accept: the capacity without the tables' spatial
order, the literal greedy as separate launches, the dense greedy's sweeps."""
import numpy as np
import pytest

from tests.test_gpu_sgs_dense_route import _sweep_bytes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def up(x):
    return (x + 255) // 256 * 256


def _bytes(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("n,nn,dtype", [(300, 8, torch.float32), (1500, 16, torch.bfloat16)])
def test_capacity_without_the_spatial_order(n, nn, dtype):
    import paper_2608_13226_amd as cp
    lib = cp.library()
    g = torch.Generator(device="cuda").manual_seed(n)
    feats = torch.randn(n, 256, device="cuda", generator=g).to(dtype)
    pos = 5.0 * torch.rand(n, 3, device="cuda", generator=g)
    frame = (torch.arange(n, device="cuda") // 100).to(torch.int32)
    # Tables, pairs, maxima, scores, partial sums.
    least = up(n * (nn + 1) * 4) + up(n * nn * 24) + 256 + up(n * 8) + up((n + 255) // 256 * 8)
    assert least < lib.coverprune_fst_capacity_workspace(n, nn)
    print(f"capacity least workspace n={n}", flush=True)
    v0, r0 = cp.fst_capacity(feats, pos, frame, nn)
    v1, r1 = cp.fst_capacity(feats, pos, frame, nn, workspace=_bytes(least))
    assert torch.equal(v0, v1) and torch.equal(r0, r1)
    with pytest.raises(cp.CoverPruneError, match="workspace"):
        cp.fst_capacity(feats, pos, frame, nn, workspace=_bytes(least - 256))


def _literal_bytes(n, k):
    """E, a, b, r, column sums, partial scores, objective shares, chosen flags."""
    kp, nrb, strips = (k + 3) // 4 * 4, (n + 63) // 64, (n + 255) // 256
    panels = max(1, min(64, (512 + strips - 1) // strips))
    return (up(n * kp * 8) + up(kp * 8) + 2 * up(n * 8) + up(nrb * kp * 8) + up(panels * n * 8) + up(nrb * 8) + up(n))


@pytest.mark.parametrize("kind", ["plain", "underflow", "unreachable", "no capacity"])
@pytest.mark.parametrize("n,k", [(65, 9), (777, 40), (2048, 70)])
def test_literal_as_separate_launches(n, k, kind):
    import paper_2608_13226_amd as cp
    lib = cp.library()
    rng = np.random.default_rng(n)
    c = (3.0 * rng.random((n, n))).astype(np.float32)
    eps = 0.05
    if kind == "underflow":
        eps = 1e-3                                  # E is 0 beyond C = 0.75
    elif kind == "unreachable":
        # A fifth of the tokens do not reach some targets: scores of infinity
        # or, with no residual there, NaN, which come after all others.
        c[(rng.random(n) < 0.2)[:, None] & (rng.random((n, n)) < 0.2)] = np.inf
    np.fill_diagonal(c, 0.0)
    v = rng.random(n).astype(np.float32)
    if kind == "no capacity":
        v[: n // 2] = 0.0
    v /= v.sum()
    cost, cap = torch.from_numpy(c).cuda().t().contiguous(), torch.from_numpy(v).cuda()
    least = _literal_bytes(n, k)
    assert least < lib.coverprune_sgs_literal_workspace(n, k)
    print(f"literal least workspace {kind} n={n}", flush=True)
    one = cp.sgs_literal_select(cost, cap, k, epsilon=eps, rounds=12)
    sep = cp.sgs_literal_select(cost, cap, k, epsilon=eps, rounds=12, workspace=_bytes(least))
    assert torch.equal(one.selected, sep.selected)
    for x, y in ((one.score, sep.score), (one.residual, sep.residual), (one.objective, sep.objective)):
        assert torch.allclose(x, y, rtol=1e-9, atol=1e-14, equal_nan=True)
    with pytest.raises(cp.CoverPruneError, match="workspace"):
        cp.sgs_literal_select(cost, cap, k, epsilon=eps, rounds=12, workspace=_bytes(least - 256))


def test_dense_greedy_when_memory_is_short(monkeypatch):
    import paper_2608_13226_amd as cp
    n, k = 1500, 40
    g = torch.Generator(device="cuda").manual_seed(1)
    cost, cap = 3.0 * torch.rand(n, n, device="cuda", generator=g), torch.rand(n, device="cuda", generator=g)
    sweeps = cp.sgs_select(cost, cap, k, c0=3.0, check=True, workspace=_bytes(_sweep_bytes(n, k)))
    real, asked = cp._workspace, []

    def short(nbytes, device):
        asked.append(nbytes)
        if nbytes > _sweep_bytes(n, k):
            raise torch.cuda.OutOfMemoryError("no room")
        return real(nbytes, device)

    monkeypatch.setattr(cp, "_workspace", short)
    print("dense greedy, short of memory", flush=True)
    r = cp.sgs_select(cost, cap, k, c0=3.0, check=True)
    assert asked[-1] == _sweep_bytes(n, k)
    for x, y in ((r.selected, sweeps.selected), (r.gain, sweeps.gain), (r.objective, sweeps.objective)):
        assert torch.equal(x, y)
    with pytest.raises(torch.cuda.OutOfMemoryError):
        cp.sgs_select(cost, cap, k, c0=3.0, incremental=True)

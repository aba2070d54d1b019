"""The literal greedy's persistent launch (n <= 2048, k <= 256) against its
separate launches, which a trajectory to follow always takes: the same
trajectory's scores, residual masses and final cost."""
import numpy as np
import pytest

from tests import parity

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _case(n, seed):
    s = parity.sample_scene("n4096_d1152", n, seed, salt=5100)
    C32 = parity.oracle_cost(s)[0].astype(np.float32)
    return torch.from_numpy(np.ascontiguousarray(C32.T)).cuda(), torch.from_numpy(s.capacity).cuda()


# Edges of the 64-row solver blocks, 8-row scoring blocks and 64-column
# chunks, the smallest and the largest scene and budget.
@pytest.mark.parametrize("n,k,rounds", [(1, 1, 3), (7, 3, 20), (64, 64, 10), (65, 20, 50), (513, 130, 10),
                                        (1000, 64, 20), (2041, 65, 5), (2048, 256, 3)])
def test_persistent_equals_separate_launches(n, k, rounds):
    import paper_2608_13226_amd as cp
    cost, cap = _case(n, n)
    print(f"literal persistent n={n} k={k} rounds={rounds}", flush=True)
    a = cp.sgs_literal_select(cost, cap, k, epsilon=0.05, rounds=rounds)
    b = cp.sgs_literal_select(cost, cap, k, epsilon=0.05, rounds=rounds, follow=a.selected)
    torch.cuda.synchronize()
    assert sorted(set(a.selected.tolist())) == sorted(a.selected.tolist()) and min(a.selected.tolist()) >= 0
    # Both sum at most 2048 nonnegative float64 terms, in another order (2048 x
    # 2^-53 = 2.3e-13 a sum), twice a round; twice that bound.
    tol = 4 * rounds * 2.3e-13 + 1e-13
    for x, y in ((a.score, b.score), (a.residual, b.residual), (a.objective, b.objective)):
        assert np.allclose(x.cpu().numpy(), y.cpu().numpy(), rtol=tol, atol=tol * float(x.abs().max()))


def test_persistent_that_gives_up(monkeypatch):
    import paper_2608_13226_amd as cp
    cost, cap = _case(300, 1)
    print("literal persistent abort path", flush=True)
    monkeypatch.setenv("COVERPRUNE_TEST_ABORT", "1")
    r = cp.sgs_literal_select(cost, cap, 20, epsilon=0.05, rounds=10)
    torch.cuda.synchronize()
    assert bool((r.selected == -1).all())
    monkeypatch.delenv("COVERPRUNE_TEST_ABORT")
    r = cp.sgs_literal_select(cost, cap, 20, epsilon=0.05, rounds=10)
    assert int(r.selected.min()) >= 0


def test_long_solves_take_the_separate_launches(monkeypatch):
    # The persistent launch's scoring blocks wait through a whole solve, so past
    # 16384 rounds the separate launches serve, which wait for nothing: a launch
    # that is made to give up at its first unmet wait tells the two apart.
    import paper_2608_13226_amd as cp
    cost, cap = _case(64, 2)
    monkeypatch.setenv("COVERPRUNE_TEST_ABORT", "1")
    for rounds in (16384, 16385):
        print(f"literal rounds={rounds}", flush=True)
        r = cp.sgs_literal_select(cost, cap, 2, epsilon=0.05, rounds=rounds)
        torch.cuda.synchronize()
        assert (int(r.selected.min()) >= 0) == (rounds > 16384)
    monkeypatch.delenv("COVERPRUNE_TEST_ABORT")
    one = cp.sgs_literal_select(cost, cap, 2, epsilon=0.05, rounds=16384)
    torch.cuda.synchronize()
    assert one.selected.tolist() == r.selected.tolist()

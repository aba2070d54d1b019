"""The capacity's neighbour tables from the spatial order (1024 tokens on):
scores against the oracle at the edges of its 64-token chunks and 8-query
blocks, on scenes that strain the bounds: a lattice full of equal distances,
a cluster of coincident tokens (rows left to the radix select), a line, two far
groups, one token far from all."""
import numpy as np
import pytest

from oracle import capacity

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _positions(kind, n, rng):
    if kind == "uniform":
        return rng.random((n, 3)) * [10, 10, 3]
    if kind == "lattice":
        return rng.integers(0, 12, (n, 3)) * 0.25
    if kind == "coincident":
        p = rng.random((n, 3)) * 4
        p[: n // 2] = [1.0, 2.0, 0.5]
        return p
    if kind == "line":
        return np.outer(rng.random(n), [100.0, 0.0, 0.0])
    if kind == "two groups":
        p = rng.normal(0, 0.01, (n, 3))
        p[n // 3:] += 1000.0
        return p
    p = rng.normal(0, 1.0, (n, 3))              # "outlier"
    p[7] = 1e6
    return p


@pytest.mark.parametrize("kind", ["uniform", "lattice", "coincident", "line", "two groups", "outlier"])
@pytest.mark.parametrize("n,nn", [(1024, 16), (1025, 1), (1091, 127), (2500, 12)])
def test_scores_from_the_spatial_order(kind, n, nn):
    import paper_2608_13226_amd as cp
    rng = np.random.default_rng(n + nn)
    pos = _positions(kind, n, rng).astype(np.float32)
    feats = rng.normal(0, 1, (n, 16)).astype(np.float32)
    frame = rng.integers(0, 9, n).astype(np.int32)
    print(f"capacity sorted {kind} n={n} nn={nn}", flush=True)
    v, r = cp.fst_capacity(torch.from_numpy(feats).cuda(), torch.from_numpy(pos).cuda(),
                           torch.from_numpy(frame).cuda(), nn)
    torch.cuda.synchronize()
    ref = capacity.capacity_ref(feats.astype(np.float64), pos, frame, nn)
    # float64 sums of float64 terms in another order.
    assert np.allclose(r.cpu().numpy(), ref["r"], rtol=1e-12, atol=1e-15)
    assert np.allclose(v.cpu().numpy(), ref["v"], rtol=2 ** -23, atol=0.0)


def _strange(kind, n, rng):
    p = rng.random((n, 3)) * [10, 10, 3]
    some = rng.choice(n, 40, replace=False)
    if kind == "nan":
        p[some, rng.integers(0, 3, 40)] = np.nan
    elif kind == "infinite":
        p[some, rng.integers(0, 3, 40)] = np.where(rng.random(40) < 0.5, np.inf, -np.inf)
    elif kind == "all nan":
        p[:] = np.nan
    elif kind == "huge":
        p[some] = rng.choice([-3.0e38, 3.0e38], (40, 3))
    else:                                        # "tiny": differences below the normal range
        p *= 1e-42
    return p.astype(np.float32)


@pytest.mark.parametrize("kind", ["nan", "infinite", "all nan", "huge", "tiny"])
@pytest.mark.parametrize("n,nn", [(1024, 16), (1091, 127), (2500, 3)])
def test_strange_positions_as_in_index_order(kind, n, nn):
    # The spatial order only leaves tokens out, so whatever a distance is, the
    # tables are those of the index order (a workspace without room for it).
    import paper_2608_13226_amd as cp
    from tests.test_gpu_workspaces import up
    rng = np.random.default_rng(n + nn)
    pos = torch.from_numpy(_strange(kind, n, rng)).cuda()
    feats = torch.from_numpy(rng.normal(0, 1, (n, 16)).astype(np.float32)).cuda()
    frame = torch.from_numpy(rng.integers(0, 9, n).astype(np.int32)).cuda()
    least = up(n * (nn + 1) * 4) + up(n * nn * 24) + 256 + up(n * 8) + up((n + 255) // 256 * 8)
    print(f"capacity sorted {kind} n={n} nn={nn}", flush=True)
    v0, r0 = cp.fst_capacity(feats, pos, frame, nn)
    v1, r1 = cp.fst_capacity(feats, pos, frame, nn, workspace=torch.empty(least, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert torch.equal(r0.view(torch.int64), r1.view(torch.int64))
    assert torch.equal(v0.view(torch.int32), v1.view(torch.int32))

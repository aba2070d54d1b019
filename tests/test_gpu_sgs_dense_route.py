"""The dense form up to 8192 tokens runs the incremental greedy when the data
lie in its fixed point's domain, and the sweeps when they do not (negative
costs, capacities of too many magnitudes, a workspace for the sweeps alone).
Either way: the oracle's picks, gains and objective."""
import numpy as np
import pytest

from oracle import sgs
from tests import parity

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _data(kind, n, rng):
    c = (3.0 * rng.random((n, n))).astype(np.float32)
    np.fill_diagonal(c, 0.0)
    v = rng.random(n).astype(np.float32)
    if kind == "negative cost":
        c[rng.integers(0, n, 20), rng.integers(0, n, 20)] = -0.25
    elif kind == "above c0":
        c[rng.random((n, n)) < 0.3] = 7.0
        c[0, :3] = np.inf
    elif kind == "tiny capacities":
        v[: n // 2] *= 1e-20
    elif kind == "zero capacities":
        v[: n // 2] = 0.0
    return c, v                                  # source-major


@pytest.mark.parametrize("kind", ["plain", "negative cost", "above c0", "tiny capacities", "zero capacities"])
@pytest.mark.parametrize("n,k", [(1, 1), (130, 130), (777, 90), (1024, 40)])
def test_dense_form_on_any_data(kind, n, k):
    import paper_2608_13226_amd as cp
    rng = np.random.default_rng(n)
    if n == 1:
        c, v = np.zeros((1, 1), np.float32), np.ones(1, np.float32)
    else:
        c, v = _data(kind, n, rng)
    print(f"sgs dense route {kind} n={n} k={k}", flush=True)
    cost = torch.from_numpy(c).cuda().t().contiguous()
    cap = torch.from_numpy(v).cuda()
    small = torch.empty(_sweep_bytes(n, k), dtype=torch.uint8, device="cuda")
    assert small.numel() < cp.library().coverprune_sgs_workspace(n, k, cp.CP_SGS_DENSE)
    full = cp.sgs_select(cost, cap, k, c0=3.0, check=True)
    C = np.where(np.isinf(c), 1e30, c).astype(np.float64)
    ref = sgs.sgs_ref(C, v.astype(np.float64), k, 3.0)
    sweeps = cp.sgs_select(cost, cap, k, c0=3.0, check=True, workspace=small)
    for r in (full, sweeps):
        sel = r.selected.cpu().numpy()
        # float32 differences of costs below 3: 2^-24 of them a term.
        tol = 3.0 * 2.0 ** -23 * float(v.sum())
        ties, g_or, o_or = parity.replay_greedy(C, v, 3.0, sel, tie_atol=tol)
        assert np.allclose(r.gain.cpu().numpy(), g_or, rtol=1e-6, atol=tol)
        assert np.allclose(r.objective.cpu().numpy(), o_or, rtol=1e-9, atol=1e-12)
        if not ties:
            assert np.array_equal(sel, ref["selected"])


def _sweep_bytes(n, k):
    """What the sweeps alone ask for: private best costs and mask, 64 panels of
    partial gains, strip winners, objective shares, keys, counters."""
    up = lambda x: (x + 255) // 256 * 256
    strips = (n + 255) // 256
    return (up(strips * (n + 64) * 4) + up(n * 4) + up(64 * n * 8) + up(1024 * 8) + up(64 * 8) + up(k * 8) +
            up(1024 * 4) + 256)

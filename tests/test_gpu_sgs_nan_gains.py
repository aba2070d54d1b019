"""Capacities that are not finite make every gain of the sweeps a NaN, and after
as many picks as there are strips of 256 columns no strip has a winner: the
picks are then unspecified, but tokens of the scene, so nothing outside the
cost is read."""
import pytest

from tests.test_gpu_sgs_dense_route import _sweep_bytes

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("n,k", [(600, 20), (2500, 30)])
def test_picks_stay_inside_the_scene(n, k, bad):
    import paper_2608_13226_amd as cp
    g = torch.Generator(device="cuda").manual_seed(n)
    cost = 3.0 * torch.rand(n, n, device="cuda", generator=g)
    cost.fill_diagonal_(0.0)
    cap = torch.rand(n, device="cuda", generator=g)
    cap[n - 1] = bad
    small = torch.empty(_sweep_bytes(n, k), dtype=torch.uint8, device="cuda")
    print(f"sgs sweeps with a capacity of {bad} n={n}", flush=True)
    for ws in (small, None):
        r = cp.sgs_select(cost, cap, k, c0=3.0, workspace=ws)
        torch.cuda.synchronize()
        assert 0 <= int(r.selected.min()) and int(r.selected.max()) < n
        assert -1 <= int(r.assign.min()) and int(r.assign.max()) < n

"""A resident plan whose tree grows stays within the server's budget, to the byte.

Dense knots in a thin background give more virtual cubes than a request's estimate counts, so the plan's
size after the build decides. The second request adds cubes to a plan that has grown for the first
one. What it holds with no limit in the way is what it needs: a budget of so many bytes serves it, one
byte less does not."""
import numpy as np
import pytest

from tests.hpmcase import log

pytestmark = pytest.mark.gpu


def _knots(torch, k):
    rng = np.random.Generator(np.random.PCG64(5))
    centre = rng.random((k, 3)) * 0.9 + 0.05
    pts = np.concatenate([rng.random((3200, 3))] + [c + 0.004 * (rng.random((66, 3)) - 0.5) for c in centre])
    x, y, z = (torch.tensor(pts[:, i], dtype=torch.float64, device="cuda") for i in range(3))
    return x, y, z, torch.full_like(x, 1.0 / len(pts))


def _serve(hpm, prob, sets, budget):
    with hpm.Server(slots=1, hbm_budget=budget) as sv:
        return [sv.wait(sv.submit(prob, *s))[0] for s in sets]


def test_grown_plan_holds_no_more_than_the_budget():
    import torch
    from paper_1906_10734_amd import hpm
    prob = hpm.Problem(ng=6, precision="f64", leaf_capacity=64, max_depth=10, softening=1e-3, m2l="cells")
    sets = [_knots(torch, k) for k in (24, 40)]
    free = _serve(hpm, prob, sets, 1 << 34)
    need = free[1]["plan_bytes"]
    log(f"[cap] estimate {free[1]['estimate_bytes']} first {free[0]['plan_bytes']} second {need}")
    assert free[1]["estimate_bytes"] < need - 1
    first, second = _serve(hpm, prob, sets, need)
    assert first["status"] == second["status"] == "HPM_OK" and second["plan_bytes"] == need
    first, second = _serve(hpm, prob, sets, need - 1)
    assert first["status"] == "HPM_OK" and second["status"] == "HPM_ERR_NO_MEMORY"

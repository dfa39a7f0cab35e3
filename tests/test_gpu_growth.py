"""Room for virtual cubes beside the cells, and the stream that only large sets need.

Dense knots of 66 particles in a thin background give far more virtual cubes than cells: 279 cells
and 1390 cubes for 12 knots (inside the room of a first build, outside that of a solve without
allocation), 462 and 2122 for 24, 707 and 2636 for 40 (outside both). A plan that was first built on
a set large enough for all of them never grows its arrays, so its results are what the grown ones
must equal: the same kernels over the same tree, whose sums do not depend on the cubes' numbers.
The bar of 1e-12 in FP64 is the one between two routes, far below what a lost cube would do."""
import numpy as np
import pytest

from tests.hpmcase import log, rel_max

pytestmark = pytest.mark.gpu


def _knots(k):
    rng = np.random.Generator(np.random.PCG64(5))
    centre = rng.random((k, 3)) * 0.9 + 0.05
    parts = [rng.random((3200, 3))] + [c + 0.004 * (rng.random((66, 3)) - 0.5) for c in centre]
    return np.concatenate(parts)


def _dev(torch, pts):
    return tuple(torch.tensor(pts[:, k], dtype=torch.float64, device="cuda") for k in range(3))


@pytest.mark.parametrize("route", ["grid", "cells"])
@pytest.mark.parametrize("knots", [12, 24, 40])
def test_grown_arrays_change_nothing(knots, route):
    import torch
    from paper_1906_10734_amd import hpm
    log(f"[growth] knots {knots} route {route}")
    prob = hpm.Problem(ng=4, precision="f64", leaf_capacity=64, max_depth=10, softening=1e-3,
                       m2l=route)
    pos = _dev(torch, _knots(knots))
    m = torch.rand(pos[0].numel(), dtype=torch.float64, device="cuda") + 0.5
    big = _dev(torch, np.random.Generator(np.random.PCG64(6)).random((1 << 17, 3)))
    roomy = hpm.Plan(prob, *big)
    roomy.rebuild(*pos)
    want = [v.cpu().numpy() for v in roomy(m)]
    fresh = hpm.Plan(prob, *pos)
    results = [fresh(m), hpm.solve(prob, *pos, m), hpm.solve_noalloc(prob, *pos, m)]
    fresh.rebuild(*big)  # past the size from which the near zone has a stream of its own
    whole = fresh(torch.ones_like(big[0]))
    roomy.rebuild(*big)
    for a, b in zip(whole, roomy(torch.ones_like(big[0]))):
        assert rel_max(a.cpu().numpy(), b.cpu().numpy()) < 1e-12
    fresh.rebuild(*pos)
    results.append(fresh(m))
    for got in results:
        for a, b in zip(got, want):
            assert rel_max(a.cpu().numpy(), b) < 1e-12

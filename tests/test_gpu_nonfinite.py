"""Masses that are infinite, or overflow, on every source-to-target route.

On a uniform tree the near zone of a leaf is the 27 leaves around it, and at every level a cube near a
target is left out of its far field. So a particle of infinite mass acts on the particles of those
27 leaves through its own pairs alone, which pull them towards it without bound, and a mass whose far
field overflows FP32 leaves its own potential as finite as the other particles make it."""
import numpy as np
import pytest

from synth import uniform_cube
from tests.hpmcase import log

pytestmark = pytest.mark.gpu

ROUTES = [("grid", 4, False), ("grid", 6, True), ("cells", 2, False), ("cells", 3, True),
          ("cells", 4, False), ("cells", 6, True), ("cells", 6, False), ("shared", 2, False),
          ("shared", 3, False), ("shared", 4, False), ("shared", 6, False)]


def _solve(p, prec, mass, at, route, ng, ext, depth=3):
    import torch
    from paper_1906_10734_amd import hpm
    dt = torch.float32 if prec == "f32" else torch.float64
    x, y, z, m = (torch.tensor(a, dtype=dt, device="cuda") for a in (p.x, p.y, p.z, p.m))
    m[at] = mass
    prob = hpm.Problem(ng=ng, precision=prec, uniform_depth=depth, softening=1e-3, m2l=route, extended=ext)
    plan = hpm.Plan(prob, x, y, z)
    out = [v.cpu().numpy() for v in plan(m)]
    plan.close()
    return out[0], np.stack(out[1:], 1)


# depth 4 at N_g = 6: enough items for the coarse split of the FP32 products
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("route,ng,ext,depth", [r + (3,) for r in ROUTES] +
                         [("cells", 6, False, 4), ("cells", 6, True, 4), ("shared", 6, False, 4)])
def test_infinite_mass_acts_on_near_targets_by_its_pairs_alone(route, ng, ext, depth, prec):
    log(f"[nonfinite] {route} ng {ng} ext {ext} {prec} depth {depth}")
    p = uniform_cube(8 ** (depth + 1), 1000).astype(np.float32)
    pos = np.stack([p.x, p.y, p.z], 1).astype(np.float64)
    leaf = (pos * 2 ** depth).astype(int)
    for at in (17, 2048):
        _, acc = _solve(p, prec, float("inf"), at, route, ng, ext, depth)
        near = np.abs(leaf - leaf[at]).max(1) <= 1
        near[at] = False
        assert near.sum() > 50
        assert (acc[near] == np.sign(pos[at] - pos[near]) * np.inf).all()
        assert np.isnan(acc[~near]).all()


@pytest.mark.parametrize("route,ng,ext", ROUTES)
def test_overflowing_mass_leaves_its_own_potential_finite(route, ng, ext):
    log(f"[overflow] {route} ng {ng} ext {ext}")
    p = uniform_cube(4096, 1000).astype(np.float32)
    phi = _solve(p, "f32", 3e38, 17, route, ng, ext)[0][17]
    alone = _solve(p, "f32", 0.0, 17, route, ng, ext)[0][17]
    assert np.isfinite(phi) and abs(phi - alone) < 1e-3 * abs(alone)

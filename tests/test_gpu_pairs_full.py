"""Sibling pairs of the padded grid on trees whose split parents have most of their children.

The pairs serve trees of at least 256 split parents with 6.0 to 6.9 children each on average. Particles
fill the first K cubes of level 3, in Morton order, of the uniform depth-4 tree: 27, 28 and 40 whole cubes
of level 2 make 247, 256 and 365 split parents. Most cubes hold 30 particles and have 7.9 children, one in
ten holds 1 to 3; with 1 to 6 in every cube the same parents have about 3.4 and are taken target by
target. The cell-by-cell route sums the same pairs: FP64 to 1e-12, FP32 to 1e-5 relative RMS."""
import numpy as np
import pytest

from tests.hpmcase import log, rel_max, rel_rms

pytestmark = pytest.mark.gpu

DEPTH = 4


def _points(cubes, sparse):
    rng = np.random.Generator(np.random.PCG64(1900 + cubes))
    k = np.arange(cubes)
    lo = np.stack([sum(((k >> (3 * b + a)) & 1) << b for b in range(3)) for a in range(3)], 1) / 8.0
    n = rng.integers(1, 7, cubes) if sparse else np.where(rng.random(cubes) < 0.1, rng.integers(1, 4, cubes), 30)
    return np.concatenate([lo[i] + rng.random((n[i], 3)) / 8.0 for i in range(cubes)])


def _solve(torch, hpm, pts, prec, ng, route, ext, strict=False):
    dt = torch.float32 if prec == "f32" else torch.float64
    x, y, z = (torch.tensor(pts[:, k], dtype=torch.float32, device="cuda").to(dt).contiguous()
               for k in range(3))
    plan = hpm.Plan(hpm.Problem(ng=ng, precision=prec, uniform_depth=DEPTH, softening=1e-3, m2l=route,
                                extended=ext), x, y, z)
    if strict:
        plan.set_fp32_strict(True)
    phi = plan(torch.full_like(x, 1.0 / len(pts)))[0].double().cpu().numpy()
    locs = [plan.locals(lvl) for lvl in range(2, DEPTH + 1)]
    info = plan.info()
    parents = sum(int(plan.cells(lvl)["split"].sum()) for lvl in range(1, DEPTH))
    plan.close()
    return phi, locs, parents, sum(info["cells_per_level"][2:]) / parents


@pytest.mark.parametrize("cubes,parents,sparse", [(216, 247, False), (224, 256, False), (320, 365, False),
                                                  (320, 365, True)])
@pytest.mark.parametrize("ng,ext", [(4, False), (4, True), (6, False), (6, True)])
def test_grid_equals_cells(ng, ext, cubes, parents, sparse):
    import torch
    from paper_1906_10734_amd import hpm
    pts = _points(cubes, sparse)
    phi, locs, found, children = _solve(torch, hpm, pts, "f64", ng, "cells", ext)
    log(f"[full pairs] ng {ng} ext {ext} parents {found} children {children:.2f}")
    assert found == parents and (children < 5.0 if sparse else children > 7.0)
    phi_g, locs_g, _, _ = _solve(torch, hpm, pts, "f64", ng, "grid", ext)
    assert rel_rms(phi_g, phi) < 1e-12
    for a, b in zip(locs_g, locs):
        assert rel_max(a, b) < 1e-12
    for strict in (False, True):
        assert rel_rms(_solve(torch, hpm, pts, "f32", ng, "grid", ext, strict)[0], phi) < 1e-5

"""The padded-grid kernel that takes two siblings at a time, around the size from which it is used.

It serves trees of at least 256 split parents; smaller ones go target by target. Particles in K cubes of
level 3 on the uniform depth-4 tree give K split parents there, with children missing in every
pattern. The cell-by-cell route sums the same pairs: FP64 agrees with it to 1e-12 in every local
potential and in the potentials, FP32 to 1e-5 relative RMS in potential (the bars between the routes
and of the FP32 paths), with and without extended gridlets and in the all-FP32 form."""
import numpy as np
import pytest

from tests.hpmcase import log, rel_max, rel_rms

pytestmark = pytest.mark.gpu

DEPTH = 4


def _points(parents):
    rng = np.random.Generator(np.random.PCG64(1700 + parents))
    cubes = rng.choice(8 ** 3, parents, replace=False)
    lo = np.stack([cubes % 8, (cubes // 8) % 8, cubes // 64], 1) / 8.0
    k = rng.integers(1, 7, parents)  # 1 .. 6 particles, so 1 .. 6 children
    return np.concatenate([lo[i] + rng.random((k[i], 3)) / 8.0 for i in range(parents)])


def _solve(torch, hpm, pts, prec, ng, route, ext, strict=False):
    dt = torch.float32 if prec == "f32" else torch.float64
    x, y, z = (torch.tensor(pts[:, k], dtype=torch.float32, device="cuda").to(dt).contiguous()
               for k in range(3))
    prob = hpm.Problem(ng=ng, precision=prec, uniform_depth=DEPTH, softening=1e-3, m2l=route,
                       extended=ext)
    plan = hpm.Plan(prob, x, y, z)
    if strict:
        plan.set_fp32_strict(True)
    phi = plan(torch.full_like(x, 1.0 / len(pts)))[0].double().cpu().numpy()
    locs = [plan.locals(lvl) for lvl in range(2, DEPTH + 1)]
    plan.close()
    return phi, locs


@pytest.mark.parametrize("parents", [150, 200, 400])
@pytest.mark.parametrize("ng,ext", [(4, False), (4, True), (6, False), (6, True)])
def test_grid_equals_cells_around_the_pair_rule(ng, ext, parents):
    import torch
    from paper_1906_10734_amd import hpm
    pts = _points(parents)
    log(f"[pairs] ng {ng} ext {ext} level-3 parents {parents}")
    phi, locs = _solve(torch, hpm, pts, "f64", ng, "cells", ext)
    phi_g, locs_g = _solve(torch, hpm, pts, "f64", ng, "grid", ext)
    assert rel_rms(phi_g, phi) < 1e-12
    for a, b in zip(locs_g, locs):
        assert rel_max(a, b) < 1e-12
    for strict in (False, True):
        phi_32, _ = _solve(torch, hpm, pts, "f32", ng, "grid", ext, strict)
        assert rel_rms(phi_32, phi) < 1e-5

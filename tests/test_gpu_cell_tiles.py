"""The matrix-core products of the cell and shared routes at the edges of their tiles.

The kernels take the split parents of a level 8 per wave and 32 or 64 per workgroup, and the modes
of a spectrum in chunks of 8 or 32, of which the last may be half full. Particles in K chosen cubes
of one level, on a uniform tree one level deeper, make K split parents there. Against the padded grid
on the same tree FP64 agrees to 1e-12 (the bar between this library's routes); FP32 to 1e-5 relative
RMS in potential with the FP64 result of the same rounded positions (the bar of the FP32 paths)."""
import numpy as np
import pytest

from tests.hpmcase import log, rel_max, rel_rms

pytestmark = pytest.mark.gpu


def _solve(torch, hpm, pts, prec, depth, ng, route, ext):
    dt = torch.float32 if prec == "f32" else torch.float64
    x, y, z = (torch.tensor(pts[:, k], dtype=torch.float32, device="cuda").to(dt).contiguous()
               for k in range(3))
    m = torch.full_like(x, 1.0 / len(pts))
    prob = hpm.Problem(ng=ng, precision=prec, uniform_depth=depth, softening=1e-3, m2l=route,
                       extended=ext)
    plan = hpm.Plan(prob, x, y, z)
    phi = plan(m)[0].double().cpu().numpy()
    locs = [plan.locals(lvl) for lvl in range(2, depth + 1)]
    plan.close()
    return phi, locs


@pytest.mark.parametrize("depth,parents,ng,ext", [
    (3, 1, 4, False), (3, 8, 6, False), (3, 9, 6, False), (3, 31, 4, True), (3, 33, 6, False),
    (3, 64, 3, False), (4, 65, 6, False), (4, 129, 4, True), (4, 512, 4, False),
])
def test_products_at_tile_edges(depth, parents, ng, ext):
    import torch
    from paper_1906_10734_amd import hpm
    rng = np.random.Generator(np.random.PCG64(900 + parents))
    side = 2 ** (depth - 1)
    cubes = rng.choice(side ** 3, parents, replace=False)
    lo = np.stack([cubes % side, (cubes // side) % side, cubes // side ** 2], 1) / side
    pts = (lo[:, None, :] + rng.random((parents, 12, 3)) / side).reshape(-1, 3)
    log(f"[tiles] depth {depth} parents {parents} ng {ng} ext {ext}")
    grid = ext is False or ng in (4, 6)
    phi, locs = _solve(torch, hpm, pts, "f64", depth, ng, "cells", ext)
    phi32, _ = _solve(torch, hpm, pts, "f32", depth, ng, "cells", ext)
    assert rel_rms(phi32, phi) < 1e-5
    if grid:
        phi_g, locs_g = _solve(torch, hpm, pts, "f64", depth, ng, "grid", ext)
        assert rel_rms(phi, phi_g) < 1e-12
        for a, b in zip(locs, locs_g):
            if np.any(b):
                assert rel_max(a, b) < 1e-12
    if not ext:
        phi_s, _ = _solve(torch, hpm, pts, "f64", depth, ng, "shared", ext)
        assert rel_rms(phi_s, phi) < 1e-12
        phi_s32, _ = _solve(torch, hpm, pts, "f32", depth, ng, "shared", ext)
        assert rel_rms(phi_s32, phi) < 1e-5

"""The FP32 cell products of small trees, whose waves take a quad of parents and one of children each.

Uniform trees with 3 to 130 filled cubes of one level, whose products have fewer items than half the
chip's CUs; cubes that hold a few particles have children missing. Against the padded grid in FP64 on the
same rounded positions (the cell route where the grid has no such gridlet), to 1e-5 relative RMS, the bar
of the FP32 paths."""
import numpy as np
import pytest

from tests.hpmcase import log, rel_rms

pytestmark = pytest.mark.gpu


def _phi(torch, hpm, pts, prec, depth, ng, route, ext):
    dt = torch.float32 if prec == "f32" else torch.float64
    x, y, z = (torch.tensor(pts[:, k], dtype=torch.float32, device="cuda").to(dt).contiguous()
               for k in range(3))
    prob = hpm.Problem(ng=ng, precision=prec, uniform_depth=depth, softening=1e-3, m2l=route, extended=ext)
    plan = hpm.Plan(prob, x, y, z)
    phi = plan(torch.full_like(x, 1.0 / len(pts)))[0].double().cpu().numpy()
    plan.close()
    return phi


@pytest.mark.parametrize("ng,ext", [(2, False), (3, False), (4, False), (4, True), (6, False), (6, True)])
@pytest.mark.parametrize("depth,parents,per", [(2, 8, 40), (3, 3, 2), (3, 4, 12), (3, 5, 12), (3, 15, 3),
                                               (3, 16, 12), (3, 17, 12), (3, 64, 30), (4, 130, 4)])
def test_small_trees(depth, parents, per, ng, ext):
    import torch
    from paper_1906_10734_amd import hpm
    rng = np.random.Generator(np.random.PCG64(700 + 10 * parents + per))
    side = 2 ** (depth - 1)
    cubes = rng.choice(side ** 3, parents, replace=False)
    lo = np.stack([cubes % side, (cubes // side) % side, cubes // side ** 2], 1) / side
    pts = (lo[:, None, :] + rng.random((parents, per, 3)) / side).reshape(-1, 3)
    log(f"[small] depth {depth} parents {parents} per {per} ng {ng} ext {ext}")
    ref = _phi(torch, hpm, pts, "f64", depth, ng, "cells" if ext and ng < 4 else "grid", ext)
    assert rel_rms(_phi(torch, hpm, pts, "f32", depth, ng, "cells", ext), ref) < 1e-5
    if not ext:
        assert rel_rms(_phi(torch, hpm, pts, "f32", depth, ng, "shared", ext), ref) < 1e-5

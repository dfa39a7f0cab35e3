"""The device-built tables, at every gridlet order, kernel and route.

With one particle on every gridlet node of every level-2 cell, the effective masses are the particle
masses and the targets are nodes, so a solve on the uniform depth-2 tree is the direct sum itself:
the fit matrix and the Green tables have to be exact. FP64 to 1e-10 of each potential and FP32 to
1e-5 relative RMS, the bars of the two paths."""
import numpy as np
import pytest

from synth import gridlet_node_lattice
from tests.hpmcase import device, log, rel_each_max, rel_rms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("ng,route,kern", [
    (2, "grid", {}), (3, "grid", {}), (4, "grid", {}), (6, "grid", {}), (8, "grid", {}),
    (3, "grid", dict(kernel="yukawa", screening=0.05)), (4, "cells", {}), (6, "cells", {}),
    (6, "cells", dict(kernel="yukawa", screening=0.05)), (2, "shared", {}), (3, "shared", {}),
])
def test_node_lattice_is_the_direct_sum(ng, route, kern, prec):
    import torch
    from paper_1906_10734_amd import hpm
    p = gridlet_node_lattice(ng, 2, seed=70 + ng).astype(np.float32 if prec == "f32" else np.float64)
    x, y, z, m = device(p, torch)
    log(f"[tables] ng {ng} {route} {prec} {kern}")
    prob = hpm.Problem(ng=ng, precision=prec, uniform_depth=2, softening=1e-3, m2l=route, **kern)
    phi = hpm.solve(prob, x, y, z, m)[0].double().cpu().numpy()
    at = torch.arange(p.n, device="cuda")
    ref = hpm.direct_sum(x, y, z, m, at, softening=1e-3, **kern)[0].cpu().numpy()
    if prec == "f64":
        assert rel_each_max(phi, ref) < 1e-10
    else:
        assert rel_rms(phi, ref) < 1e-5

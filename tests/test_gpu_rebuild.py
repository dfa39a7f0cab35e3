"""A set rebuilt in place: the second build sizes its hash tables and its near lists' chunks by what the
first one found (more cells and cubes than the arrays' capacity), which must change nothing.

262,144 clustered particles with leaves of 16 make 61 k cells, and more cubes than the 98 k cells that
the capacity allows for; near-list chunks are then 16 leaves instead of 8. FP64, the same sums: 1e-12."""
import pytest

from synth import clustered_spheres
from tests.hpmcase import device, log, rel_max

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf", [(262144, 16), (2000, 16)])
def test_second_build_equals_the_first(n, leaf):
    import torch
    from paper_1906_10734_amd import hpm
    log(f"[rebuild] {n} leaf {leaf}")
    x, y, z, m = device(clustered_spheres(n, 13), torch)
    plan = hpm.Plan(hpm.Problem(ng=2, precision="f64", leaf_capacity=leaf, softening=1e-3), x, y, z)
    first, info = [v.cpu().numpy() for v in plan(m)], plan.info()
    for _ in range(2):
        plan.rebuild(x, y, z)
        again = plan.info()
        assert all(again[k] == info[k] for k in info if k != "device_bytes")
        for a, b in zip(plan(m), first):
            assert rel_max(a.cpu().numpy(), b) < 1e-12
    plan.close()

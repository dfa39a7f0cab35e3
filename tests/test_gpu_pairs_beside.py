"""FP64, N_g = 4 with extended gridlets: target by target where the near zone runs beside the grid
kernel and the tree is of medium size, in sibling pairs where it does not. A target gets the same
operations in the same order from either kernel, so the results are the same bits."""
import pytest

from synth import plummer_sphere
from tests.hpmcase import device, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65535, 66001, 150001])
def test_near_zone_beside_or_in_line_gives_the_same_bits(n):
    import torch
    from paper_1906_10734_amd import hpm
    log(f"[pairs beside] {n}")
    x, y, z, m = device(plummer_sphere(n, 11, a=0.1), torch)
    plan = hpm.Plan(hpm.Problem(ng=4, precision="f64", extended=True, leaf_capacity=64, softening=1e-3),
                    x, y, z)
    beside = plan(m)
    plan.set_overlap(False)
    for a, b in zip(beside, plan(m)):
        assert torch.equal(a, b)
    plan.close()

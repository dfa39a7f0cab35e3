"""The particle order at the edges of the sort's waves, rounds, batches and tiles, and on either side
of the tile sizes' rule: exactly numpy's stable order of the Morton keys, with few distinct keys (long
runs of one digit) and with many."""
import numpy as np
import pytest

from oracle.tree import cell_index, morton_key
from tests.hpmcase import log

pytestmark = pytest.mark.gpu

SIZES = [1, 63, 65, 256, 257, 1023, 1024, 1025, 5000, (1 << 19) - 1, 1 << 19, (1 << 19) + 1,
         (1 << 19) + 4097]


@pytest.mark.parametrize("depth", [2, 10])
@pytest.mark.parametrize("n", SIZES)
def test_order_is_the_stable_order_of_the_keys(n, depth):
    import torch
    from paper_1906_10734_amd import hpm
    log(f"[sort] n {n} depth {depth}")
    pts = np.random.Generator(np.random.PCG64(n)).random((n, 3)) ** 2
    pos = [torch.tensor(pts[:, k], dtype=torch.float64, device="cuda") for k in range(3)]
    prob = hpm.Problem(ng=2, precision="f64", leaf_capacity=64, max_depth=depth, softening=1e-3)
    q = cell_index(pts, (0.0, 0.0, 0.0), 1.0, depth)
    key = morton_key(q[:, 0], q[:, 1], q[:, 2], depth)
    plan = hpm.Plan(prob, *pos)
    assert np.array_equal(plan.perm(), np.argsort(key, kind="stable"))

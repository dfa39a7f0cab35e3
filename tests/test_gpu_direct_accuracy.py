"""The device direct sum against 80-bit sums, at every target count that changes its launch.

Each of a thread's sums has at most n / 256 terms and the rest are pairwise or compensated, so what is
left is about the result's own rounding: the error's RMS over 100 targets, relative to the potentials',
below one rounding, 2^-53, and four for the accelerations, whose terms cancel."""
import numpy as np
import pytest

from synth import clustered_spheres, plummer_sphere, uniform_cube
from tests.hpmcase import device, log

pytestmark = pytest.mark.gpu


def _exact(p, at, eps):
    x, y, z, m = (np.asarray(a, np.longdouble) for a in (p.x, p.y, p.z, p.m))
    out = np.zeros((4, len(at)), np.longdouble)
    for k, t in enumerate(at):
        d = [c[t] - c for c in (x, y, z)]
        r2 = d[0] ** 2 + d[1] ** 2 + d[2] ** 2 + np.longdouble(eps) ** 2
        w = m / np.sqrt(r2)
        w[t] = 0
        out[:, k] = [-w.sum()] + [-(w / r2 * c).sum() for c in d]
    return out


@pytest.mark.parametrize("gen", [plummer_sphere, uniform_cube, clustered_spheres])
@pytest.mark.parametrize("nt", [100, 511, 512, 2048, 4096])
def test_error_is_one_rounding(gen, nt):
    import torch
    from paper_1906_10734_amd import hpm
    p = gen(16384, 5)
    x, y, z, m = device(p, torch)
    at = np.random.default_rng(1).permutation(16384)[:nt]
    got = np.stack([v.cpu().numpy()[:100] for v in
                    hpm.direct_sum(x, y, z, m, torch.tensor(at, device="cuda"), 1.0, 1e-3)])
    want = _exact(p, at[:100], 1e-3)
    err = got.astype(np.longdouble) - want
    phi = float(np.sqrt((err[0] ** 2).sum() / (want[0] ** 2).sum()))
    acc = float(np.sqrt((err[1:] ** 2).sum() / (want[1:] ** 2).sum()))
    log(f"[direct accuracy] {gen.__name__} targets {nt}: phi {phi:.2e} acc {acc:.2e}")
    assert phi < 2.0 ** -53 and acc < 2.0 ** -51


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_a_particle_alone_feels_nothing(value):
    import torch
    from paper_1906_10734_amd import hpm
    x = torch.full((1,), value, dtype=torch.float64, device="cuda")
    y = torch.full_like(x, 0.5)
    out = hpm.direct_sum(x, y, y, y, torch.tensor([0], device="cuda"))
    assert all(float(v[0]) == 0.0 for v in out)

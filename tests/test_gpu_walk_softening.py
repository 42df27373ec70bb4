"""Softenings at the ends of what tb_gravity accepts (any finite eps >= 0): eps^2 infinite,
barely finite, below the smallest normal number, and zero.  Every cell is opened, so the
reference is the direct sum in 64 bits."""
import numpy as np
import pytest
import torch

from paper_2312_06102_amd import datagen as dg
from paper_2312_06102_amd import treebuild as tb

pytestmark = pytest.mark.gpu

TOL = 1e-12  # as test_gpu_gravity: of the sum of the terms' magnitudes


@pytest.mark.parametrize("eps", [1.7e308, 1e200, 1.35e154, 1e154, 1e100, 1e-100, 1e-153, 1e-160,
                                 1e-165, 0.0])
@pytest.mark.parametrize("n_crit", [16, 300])
def test_direct_sum(eps, n_crit):
    n = 700
    pos, mass = dg.plummer(n, seed=77, masses="lognormal")
    b = tb.Builder(n, 8, sorted_particles=True)
    b.launch(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), ((0, 0, 0), 1.0))
    b.result()
    acc = b.gravity(0.0, n_crit, eps, True)[0].cpu().numpy()
    x = pos[b.out.perm.cpu().numpy()].astype(np.float64)
    m = mass[b.out.perm.cpu().numpy()].astype(np.float64)
    d = x[:, None, :] - x[None, :, :]
    with np.errstate(over="ignore", under="ignore", divide="ignore"):
        s = np.sqrt((d * d).sum(2) + np.float64(eps) * np.float64(eps))
        np.fill_diagonal(s, np.inf)
        phi = -(m / s).sum(1)
        f = m / s / s / s
        want = -(f[:, :, None] * d).sum(1)
        size = (f * np.sqrt((d * d).sum(2))).sum(1)
    assert np.all(np.abs(acc[:, 3] - phi) <= TOL * np.abs(phi)), eps
    # (below 2^-1022 products lose digits: one unit of the smallest number a term)
    assert np.all(np.linalg.norm(acc[:, :3] - want, axis=1) <= TOL * size + n * 5e-324), eps


def test_coincident_pair_with_a_subnormal_square():
    """Two particles at one point and eps^2 = 1e-320: each meets the other at distance eps."""
    n, eps = 300, 1e-160
    pos, mass = dg.uniform(n, seed=62)
    pos[7] = pos[123]
    b = tb.Builder(n, 8, sorted_particles=True)
    b.launch(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), ((0, 0, 0), 1.0))
    b.result()
    phi = b.gravity(0.75, 64, eps, True)[0].cpu().numpy()[:, 3]
    perm = b.out.perm.cpu().numpy()
    s = np.sqrt(np.float64(eps) * np.float64(eps))
    for i, j in ((7, 123), (123, 7)):
        want = -np.float64(mass[j]) / s
        assert abs(phi[perm == i][0] - want) <= 1e-14 * abs(want)
    assert np.all(np.isfinite(phi))

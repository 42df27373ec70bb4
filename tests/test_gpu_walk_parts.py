"""The walk's split of a group over lanes and items of work, at the edges of both.

A group's particles are spread over lanes in sets, and large groups are cut into
parts of 32, 64 or 128 particles (by the size of the set).  Each case is compared
with the CPU walk as in test_gpu_gravity: equal lists, accelerations to 1e-12 of
the sum of the terms' magnitudes.
"""
import numpy as np
import pytest
import torch

from paper_2312_06102_amd import datagen as dg
from paper_2312_06102_amd import treebuild as tb

from test_gpu_gravity import compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 255, 256, 257, 1025])
def test_one_group_of_n(n):
    """The root is the only group: n particles on the list of all n."""
    pos, mass = dg.uniform(n, seed=60 + n)
    compare(pos, mass, 4, 0.75, 2000, 1e-3, True)


@pytest.mark.parametrize("n,n_crit,quad", [(32767, 200, True), (32768, 200, False),
                                           (40000, 1000, True)])
def test_parts_of_each_size(n, n_crit, quad):
    pos, mass = dg.plummer(n, seed=61, masses="lognormal")
    compare(pos, mass, 10, 0.9, n_crit, 1e-4, quad)


def test_coincident_particles_without_softening():
    """Two particles at one point and no softening: their potentials are -inf and
    their accelerations not a number; the others are as ever."""
    pos, mass = dg.uniform(300, seed=62)
    pos[7] = pos[123]
    b = tb.Builder(300, 8, sorted_particles=True)
    b.launch(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), ((0, 0, 0), 1.0))
    b.result()
    acc = b.gravity(0.75, 64, 0.0, True)[0].cpu().numpy()
    perm = b.out.perm.cpu().numpy()
    hit = np.isin(perm, (7, 123))
    assert np.all(np.isneginf(acc[hit, 3])) and np.all(np.isnan(acc[hit, :3]))
    assert np.all(np.isfinite(acc[~hit]))

"""tb_gravity with a c_max below the number of particles, as a caller that passes its tree's
number of cells has it: the walk stays inside its workspace and gives the same forces."""
import numpy as np
import pytest
import torch

import oracle
from paper_2312_06102_amd import datagen as dg
from paper_2312_06102_amd import treebuild as tb

pytestmark = pytest.mark.gpu

GUARD = 1 << 16
TOL = 1e-12  # as test_gpu_gravity: of the sum of the terms' magnitudes


@pytest.mark.parametrize("n,n_leaf,n_crit,coincident", [
    (1 << 14, 512, 64, 0),        # few cells, groups of hundreds
    (1 << 14, 1024, 5000, 0),     # groups of more than one pass
    (5000, 256, 256, 3000),       # a leaf of more than one pass
    (40_000, 300, 512, 0),
    (300, 1024, 1, 0)])           # the root is a leaf
@pytest.mark.parametrize("spare", [0, 7])
def test_workspace_of_the_trimmed_tree(n, n_leaf, n_crit, coincident, spare):
    pos, mass = dg.plummer(n, seed=n + n_leaf, masses="lognormal")
    pos[:coincident] = pos[0]
    b = tb.Builder(n, n_leaf, sorted_particles=True)
    b.launch(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), ((0, 0, 0), 1.0))
    c_max = b.result()["n_cells"] + spare
    assert c_max < n
    ws_bytes = tb.tb_gravity_workspace_bytes(c_max)
    ws = torch.full((ws_bytes + GUARD,), 0x5A, dtype=torch.uint8, device="cuda")
    acc = torch.zeros((n, 4), dtype=torch.float64, device="cuda")
    stats = torch.zeros(2, dtype=torch.int64, device="cuda")
    rc = tb.tb_gravity(b.out.pos_sorted.data_ptr(), b.out.mass_sorted.data_ptr(), n, b._struct,
                       c_max, 0.75, n_crit, 1e-3, tb.TB_GRAV_QUADRUPOLE, acc.data_ptr(),
                       stats.data_ptr(), ws.data_ptr(), ws_bytes,
                       torch.cuda.current_stream().cuda_stream)
    assert rc == tb.TB_OK
    torch.cuda.synchronize()
    assert bool((ws[ws_bytes:] == 0x5A).all())
    t = oracle.build(pos, mass, n_leaf)
    o, ost = oracle.walk_forces(pos, mass, t, theta=0.75, n_crit=n_crit, eps=1e-3,
                                quadrupole=True)
    assert stats.cpu().tolist() == [ost["groups"], ost["interactions"]]
    g = acc.cpu().numpy()
    assert np.all(np.linalg.norm(g[:, :3] - o[:, :3], axis=1) <= TOL * o[:, 4])
    assert np.all(np.abs(g[:, 3] - o[:, 3]) <= TOL * np.abs(o[:, 3]))

"""A set's tree in a batch is its standalone tree bit for bit, also where the two take other
kernels: a batch above 786432 particles has cell tiles of 2048 and, for n_leaf 4 and 5, the
parents of one launch a depth, its smaller sets alone tiles of 512 and the parents by their
tiles."""
import numpy as np
import pytest
import torch

from paper_2312_06102_amd import datagen as dg
from paper_2312_06102_amd import treebuild as tb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("curve", ["morton", "hilbert"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n_leaf", [1, 4, 5, 6, 16])
def test_set_alone_and_in_a_large_batch(n_leaf, precision, curve):
    sizes = np.array([5000, 1, 300_000, 17, 500_000, 60_000, 513], np.int64)
    pos, mass, off = dg.batched_plummer(sizes, seed=n_leaf)
    rng = np.random.default_rng(n_leaf)
    mass = (mass * np.exp(rng.normal(0.0, 1.0, mass.size))).astype(np.float32)
    r = tb.build_batched(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(),
                         torch.from_numpy(off).cuda(), n_leaf, precision=precision, curve=curve)
    co = r["cell_offsets"].cpu().numpy()
    for b in range(sizes.size):
        s = slice(int(off[b]), int(off[b + 1]))
        one = tb.build(torch.from_numpy(pos[s].copy()).cuda(),
                       torch.from_numpy(mass[s].copy()).cuda(), n_leaf, precision=precision,
                       curve=curve)
        c = slice(int(co[b]), int(co[b + 1]))
        for k in ("cell_key", "cell_level", "cell_count", "com", "quad"):
            assert torch.equal(r[k][c], one[k]), (b, k, int((r[k][c] != one[k]).sum()))

"""Batches whose sets lie over the ends of groups of tiles (32, 1024): tiles are counted
through all the sets, so a small set may begin in one group and end in the next.  Every
set's cells against the set's own build, with the outputs holding other values before."""
import numpy as np
import pytest
import torch

from paper_2312_06102_amd import datagen as dg
from paper_2312_06102_amd import treebuild as tb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes", [
    [10] * 31 + [1000],                              # tiles of 512: the last set over tile 32
    [10] * 1023 + [1000, 40],                        # over tile 1024, fewer than 32 tiles' particles
    [100] * 1023 + [30_000, 40],                     # fewer than 1024 tiles' particles
    [500] * 1020 + [400_000, 7],                     # tiles of 2048
], ids=["tile32", "tile1024", "tile1024_two_levels", "large_tiles"])
def test_sets_over_the_ends_of_groups(sizes, precision):
    sizes = np.array(sizes, np.int64)
    pos, mass, off = dg.batched_plummer(sizes, seed=int(sizes.size))
    b = tb.BatchBuilder(int(off[-1]), sizes.size, 16, precision)
    for k in ("com", "quad"):
        getattr(b.out, k).fill_(float("nan"))
    for k in ("cell_count", "child_ptr"):
        getattr(b.out, k).fill_(-77)
    b.launch(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(),
             torch.from_numpy(off).cuda())
    r = b.result()
    co = r["cell_offsets"].cpu().numpy()
    for s in sorted({0, 30, sizes.size // 2, sizes.size - 3, sizes.size - 2, sizes.size - 1}):
        if s >= sizes.size:
            continue
        at = slice(int(off[s]), int(off[s + 1]))
        one = tb.build(torch.from_numpy(pos[at].copy()).cuda(),
                       torch.from_numpy(mass[at].copy()).cuda(), 16, precision=precision)
        c = slice(int(co[s]), int(co[s + 1]))
        for k in ("cell_key", "cell_count", "com", "quad"):
            assert torch.equal(r[k][c], one[k]), (s, k)
        kids = r["child_ptr"][c].clone()
        kids[:, 0] -= (kids[:, 0] >= 0).int() * int(co[s])
        assert torch.equal(kids, one["child_ptr"]), s

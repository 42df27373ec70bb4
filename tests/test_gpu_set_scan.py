"""The scan over the sets of a batch in one wave (64 sets), workgroups of 64 (up to 1024)
and of 256: batches on both sides of each limit against each set's own build."""
import numpy as np
import pytest
import torch

from paper_2312_06102_amd import datagen as dg
from paper_2312_06102_amd import treebuild as tb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nsets", [63, 64, 65, 128, 129, 1023, 1024, 1025, 1281])
def test_set_offsets(nsets):
    rng = np.random.default_rng(nsets)
    sizes = rng.integers(0, 60, nsets).astype(np.int64)
    pos, mass, off = dg.batched_plummer(sizes, seed=nsets)
    r = tb.build_batched(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(),
                         torch.from_numpy(off).cuda(), 4)
    co, lo = r["cell_offsets"].cpu().numpy(), r["level_offset"].cpu().numpy()
    assert co[0] == 0 and co[-1] == r["n_cells"]
    for b in range(0, nsets, max(1, nsets // 40)):
        if sizes[b] == 0:
            assert co[b + 1] == co[b]
            continue
        s = slice(int(off[b]), int(off[b + 1]))
        one = tb.build(torch.from_numpy(pos[s].copy()).cuda(),
                       torch.from_numpy(mass[s].copy()).cuda(), 4)
        assert co[b + 1] - co[b] == one["n_cells"], b
        assert np.array_equal(lo[b] - co[b], one["level_offset"].cpu().numpy()), b
        assert torch.equal(r["cell_key"][int(co[b]):int(co[b + 1])], one["cell_key"]), b

"""Leaves of more than 95 particles: the radix passes sort every key bit, with whole keys
and their indices side by side in the first passes, and leave their order in perm.  Sizes at
which the formats change, every mode of the sort, and batches, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2312_06102_amd import datagen as dg
from paper_2312_06102_amd import treebuild as tb

from test_gpu_runs import check, clumps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [97, 8192, 8193, 2 ** 17, 2 ** 17 + 1, 2 ** 20 + 1, 3_000_000])
@pytest.mark.parametrize("n_leaf", [96, 128, 1024])
def test_sizes(n, n_leaf):
    if n > 2 ** 20 and n_leaf == 1024:
        pytest.skip("two values of n_leaf are enough at these sizes")
    check(clumps(n, [min(n, 40)] * max(1, n // 4000), n + n_leaf, same=5), n_leaf)


@pytest.mark.parametrize("n", [300, 1024, 1025, 2 ** 16 + 1, 2 ** 19 + 1])
@pytest.mark.parametrize("mode", [dict(counted=True), dict(lookback=True), dict(sort_config=4),
                                  dict(sort_config=4, counted=True), dict(sort_config=5),
                                  dict(subtrees=True), dict(precision="mixed")])
def test_modes(n, mode):
    check(clumps(n, [50] * (n // 5000), n, same=9), 100, **mode)


@pytest.mark.parametrize("bits", [0, 16])
@pytest.mark.parametrize("counted", [False, True])
def test_batch(bits, counted):
    sizes = np.array([5000, 0, 1, 65_536, 97, 300, 96, 40_000, 3], np.int64)
    pos, mass, off = dg.batched_plummer(sizes, seed=12)
    boxes = np.tile(np.array([0.0, 0.0, 0.0, 1.0]), (sizes.size, 1))
    r = tb.build_batched(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(),
                         torch.from_numpy(off).cuda(), 128, torch.from_numpy(boxes).cuda(),
                         set_index_bits=bits, counted=counted)
    perm, first = r["perm"].cpu().numpy(), r["cell_first"].cpu().numpy()
    co = r["cell_offsets"].cpu().numpy()
    for b, n in enumerate(sizes):
        if n == 0:
            continue
        s = slice(int(off[b]), int(off[b + 1]))
        ref = oracle.build(pos[s], mass[s], 128, moments=False)
        assert np.array_equal(perm[s] - off[b], ref["perm"]), b
        assert co[b + 1] - co[b] == ref["n_cells"]
        assert np.array_equal(first[co[b]:co[b + 1]] - off[b], ref["cell_first"])

"""Radix tiles of 2048, 4096 and 5632 keys: sizes on both sides of each limit and at the
edges of tiles, single sets and batches, data sorted by all key bits as well; the order
exactly against the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2312_06102_amd import datagen as dg
from paper_2312_06102_amd import treebuild as tb

from test_gpu_parity import compare_structure, gpu_build

pytestmark = pytest.mark.gpu

BOX = ((0.0, 0.0, 0.0), 1.0)


@pytest.mark.parametrize("n", [2047, 2048, 2049, 4097, 2 ** 17, 2 ** 17 + 1, 33 * 4096,
                               33 * 4096 + 1, 2 ** 20, 2 ** 20 + 1])
def test_edges(n):
    pos, mass = dg.plummer(n, seed=n % 1000)
    compare_structure(gpu_build(pos, mass, 16, BOX), oracle.build(pos, mass, 16))


@pytest.mark.parametrize("n", [3000, 2 ** 17, 140_000])
@pytest.mark.parametrize("n_leaf", [16, 200])
def test_every_key_bit(n, n_leaf):
    """All in one cell of depth 14 (the sample asks for the low bits), or leaves too large
    to finish the order in the reorder."""
    rng = np.random.default_rng(n)
    pos = (0.3 + 2.0 ** -14 * rng.random((n, 3))).astype(np.float32)
    mass = np.ones(n, np.float32)
    compare_structure(gpu_build(pos, mass, n_leaf, BOX), oracle.build(pos, mass, n_leaf))


@pytest.mark.parametrize("total,small", [(2 ** 17, 0), (2 ** 17 + 7, 0), (2 ** 19, 400),
                                         (2 ** 19 + 1, 400), (2 ** 20 + 1, 0)])
def test_batches(total, small):
    """(small: sets of a few particles, which lower the mean size of a set)"""
    sizes = np.array([2048, 1, 2049, 0, 4097, 5632, 40_000] + [3] * small, np.int64)
    sizes = np.append(sizes, total - sizes.sum())
    pos, mass, off = dg.batched_plummer(sizes, seed=3)
    boxes = torch.tensor([[0.0, 0.0, 0.0, 1.0]] * len(sizes), dtype=torch.float64, device="cuda")
    r = tb.build_batched(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(),
                         torch.from_numpy(off).cuda(), 16, boxes)
    perm, keys = r["perm"].cpu().numpy(), r["cell_key"].cpu().numpy()
    co = r["cell_offsets"].cpu().numpy()
    for b, n in enumerate(sizes):
        if n == 0:
            continue
        s = slice(int(off[b]), int(off[b + 1]))
        o = oracle.build(pos[s], mass[s], 16)
        assert np.array_equal(perm[s] - int(off[b]), o["perm"]), b
        assert np.array_equal(keys[co[b]:co[b + 1]], o["cell_key"]), b


@pytest.mark.parametrize("n_leaf", [1, 16, 200])
@pytest.mark.parametrize("n", [1, 2, 33, 64, 1023, 1024, 1025, 2048, 2049, 4095, 4096, 4097,
                               8191, 8192, 8193])
def test_one_workgroup(n, n_leaf):
    pos, mass = dg.clustered(n, seed=n, n_halos=3)
    compare_structure(gpu_build(pos, mass, n_leaf, BOX), oracle.build(pos, mass, n_leaf))


@pytest.mark.parametrize("run", [32, 33, 34, 1000])
def test_one_workgroup_runs(run):
    """Runs that agree in the upper 32 key bits: the longest that the reorder finishes, and
    longer ones, among spread particles."""
    rng = np.random.default_rng(run)
    near = 0.5 + 2.0 ** -13 * rng.random((run, 3))
    pos = np.concatenate([rng.random((1500, 3)) * 0.4, near]).astype(np.float32)
    pos = pos[rng.permutation(len(pos))]
    mass = np.ones(len(pos), np.float32)
    compare_structure(gpu_build(pos, mass, 8, BOX), oracle.build(pos, mass, 8))

"""Parents built by the owners of their particles: tiles of 512 or 2048, groups of 32
tiles, groups of groups.  Sizes at the edges of each, both sides of the rule that picks this
path, precisions and curves, and batches whose sets straddle groups; structure exactly
and moments to the suite's tolerances against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2312_06102_amd import datagen as dg
from paper_2312_06102_amd import treebuild as tb

from test_gpu_parity import compare_structure, gpu_build, moment_errors

pytestmark = pytest.mark.gpu

BOX = ((0.0, 0.0, 0.0), 1.0)


def check(pos, mass, n_leaf, precision="fp64"):
    g = gpu_build(pos, mass, n_leaf, BOX, precision=precision)
    o = oracle.build(pos, mass, n_leaf)
    compare_structure(g, o)
    errs = moment_errors(g["com"].astype(np.float64), g["quad"].astype(np.float64), o["com"],
                         o["quad"], o["cell_level"])
    assert max(errs) <= (1e-12 if precision == "fp64" else 1e-5), errs


@pytest.mark.parametrize("n", [2, 17, 511, 512, 513, 2047, 2048, 2049, 4097, 16383, 16384, 16385,
                               65535, 65536, 65537, 131073, 524289, 3 * 2 ** 18,
                               3 * 2 ** 18 + 1, 2 ** 21, 2 ** 21 + 1])
def test_edges_of_tiles_and_groups(n):
    pos, mass = dg.plummer(n, seed=n, masses="lognormal")
    check(pos, mass, 16)


@pytest.mark.parametrize("n_leaf", [1, 3, 4, 5, 6, 7, 95, 96])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_both_paths(n_leaf, precision):
    pos, mass = dg.clustered(70_001, seed=n_leaf, n_halos=50, masses="lognormal")
    check(pos, mass, n_leaf, precision)


@pytest.mark.parametrize("n_leaf", [5, 6])
def test_both_paths_large_tiles(n_leaf):
    pos, mass = dg.clustered(3 * 2 ** 18 + 1, seed=n_leaf, n_halos=50, masses="lognormal")
    check(pos, mass, n_leaf)


def test_chains_of_single_children():
    """Close pairs in otherwise empty cells: parents with one child at many depths, most
    of them reaching over a tile's or a group's end."""
    rng = np.random.default_rng(3)
    base = rng.random((40_000, 3)).astype(np.float32)
    pos = np.concatenate([base, np.clip(base + np.float32(2.0 ** -19), 0, dg.F32_BELOW_ONE)])
    mass = np.full(pos.shape[0], 1.0, np.float32)
    check(pos, mass, 6)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_batch_sets_across_groups(precision):
    """Tiles of many sets in one group of tiles, and sets over several groups."""
    sizes = np.array([17] * 40 + [70_000, 1, 0, 65_536, 2049, 3] + [300] * 20 + [140_001, 5],
                     np.int64)
    pos, mass, off = dg.batched_plummer(sizes, seed=8)
    r = tb.build_batched(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(),
                         torch.from_numpy(off).cuda(), 16, precision=precision)
    co = r["cell_offsets"].cpu().numpy()
    for b, n in enumerate(sizes):
        if n == 0:
            continue
        s = slice(int(off[b]), int(off[b + 1]))
        one = tb.build(torch.from_numpy(pos[s].copy()).cuda(),
                       torch.from_numpy(mass[s].copy()).cuda(), 16, precision=precision)
        c = slice(int(co[b]), int(co[b + 1]))
        for k in ("cell_key", "cell_count", "com", "quad"):
            assert torch.equal(r[k][c], one[k]), (b, k)
        kids = r["child_ptr"][c].clone()
        kids[:, 0] -= (kids[:, 0] >= 0).int() * int(co[b])
        assert torch.equal(kids, one["child_ptr"]), b

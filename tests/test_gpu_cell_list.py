"""Tiles whose cells are listed before they are written (at most as many cells as the tile
has places) and tiles with more cells, whose threads write their own; structure exactly and
moments to the suite's tolerances against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2312_06102_amd import datagen as dg

from test_gpu_parity import compare_structure, gpu_build, moment_errors

pytestmark = pytest.mark.gpu

BOX = ((0.0, 0.0, 0.0), 1.0)


def check(pos, mass, n_leaf, precision):
    o = oracle.build(pos, mass, n_leaf)
    g = gpu_build(pos, mass, n_leaf, BOX, precision=precision)
    compare_structure(g, o)
    errs = moment_errors(g["com"].astype(np.float64), g["quad"].astype(np.float64), o["com"],
                         o["quad"], o["cell_level"])
    assert max(errs) <= (1e-12 if precision == "fp64" else 1e-5), errs
    return o


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,seed,cells", [(338, 0, 511), (341, 0, 512), (334, 3, 513)])
def test_as_many_cells_as_places(n, seed, cells, precision):
    pos, mass = dg.plummer(n, seed=seed)
    o = check(pos, mass, 1, precision)
    assert len(o["cell_key"]) == cells


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n_leaf", [1, 2, 3])
def test_tiles_on_both_sides(n_leaf, precision):
    """Tiles of 2048: over 3000 cells each, 2008 to 2191, and under 1800."""
    n = 3 * 2 ** 18 + 1
    pos, mass = dg.plummer(n, seed=2, masses="lognormal")
    o = check(pos, mass, n_leaf, precision)
    cells = np.bincount(o["cell_first"] // 2048)[:-1]
    if n_leaf == 2:
        assert cells.min() <= 2048 < cells.max()
    else:
        assert (cells.min() > 2048) == (n_leaf == 1)


def test_chains_to_the_last_depth():
    """Pairs that share every key bit but the last few: more cells than particles."""
    rng = np.random.default_rng(5)
    base = rng.random((3000, 3)).astype(np.float32)
    pos = np.concatenate([base, base + np.float32(2.0 ** -20)])
    pos = np.minimum(pos, dg.F32_BELOW_ONE).astype(np.float32)
    check(pos, np.ones(len(pos), np.float32), 1, "fp64")

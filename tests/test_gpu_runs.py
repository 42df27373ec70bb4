"""Particles that agree in the key bits the radix passes sort (the upper 32 or 40
of 63): the reorder orders runs of up to 32, k_sort_runs longer ones, and a sample of
the keys turns on the passes over the low bits for data that crowds.  Every build is
compared with the oracle: perm, keys and all cells exactly."""
import numpy as np
import pytest
import torch

import oracle
from paper_2312_06102_amd import treebuild as tb

pytestmark = pytest.mark.gpu

CELL = 2.0 ** -13  # a depth-13 cell: 39 upper key bits


def check(pos, n_leaf=16, **kw):
    mass = np.full(pos.shape[0], 1.0 / pos.shape[0], np.float32)
    r = tb.build(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), n_leaf,
                 ((0, 0, 0), 1.0), sorted_keys=True, sorted_particles=True, **kw)
    ref = oracle.build(pos, mass, n_leaf, moments=False)
    assert r["n_cells"] == ref["n_cells"]
    assert np.array_equal(r["perm"].cpu().numpy(), ref["perm"])
    assert np.array_equal(r["cell_key"].cpu().numpy().view(np.uint64), ref["cell_key"])
    for k in ("cell_level", "cell_first", "cell_count", "child_ptr"):
        assert np.array_equal(r[k].cpu().numpy(), ref[k]), k
    assert np.array_equal(r["pos_sorted"].cpu().numpy(), pos[ref["perm"]])


def clumps(n, sizes, seed, cell=CELL, same=0):
    """Uniform particles with clumps of the given sizes, each inside one small cell;
    `same` of a clump's particles coincide."""
    rng = np.random.default_rng(seed)
    pos = rng.random((n, 3), dtype=np.float32)
    at = 0
    for k, size in enumerate(sizes):
        corner = np.floor(rng.random(3) / cell) * cell
        pos[at:at + size] = corner + cell * rng.random((size, 3)) * 0.999
        pos[at:at + min(same, size)] = pos[at]
        at += size
    return pos[rng.permutation(n)]


@pytest.mark.parametrize("size", [2, 3, 31, 32, 33, 34, 64, 65, 255, 256, 257, 600])
def test_runs_around_the_cap(size):
    """Many runs of one size, so that some meet the edges of tiles and windows; few
    enough of the particles that the sample does not ask for the low passes."""
    n = 300_000 if size < 100 else 600_000
    check(clumps(n, [size] * max(1, n // (100 * size)), size))


@pytest.mark.parametrize("n_leaf", [1, 16, 95, 96, 500, 1024])
def test_runs_and_leaf_capacity(n_leaf):
    check(clumps(280_000, [20] * 100 + [50] * 40 + [3000], n_leaf, same=7), n_leaf)


@pytest.mark.parametrize("n", [33, 34, 100, 2047, 2048, 2049, 4096, 4097, 20_000, 300_000])
def test_one_run_of_everything(n):
    """All particles in one depth-14 cell, and all at one point."""
    rng = np.random.default_rng(n)
    check((0.5 + 2.0 ** -14 * rng.random((n, 3))).astype(np.float32))
    if n <= 4097:
        check(np.full((n, 3), 0.3, np.float32))


@pytest.mark.parametrize("n", [2 ** 18, 2 ** 18 + 1])
@pytest.mark.parametrize("mode", [dict(), dict(counted=True), dict(lookback=True),
                                  dict(sort_config=4), dict(curve="hilbert", sort_config=4)])
def test_every_sort_on_both_sides_of_a_width(n, mode):
    if mode.get("curve"):
        pytest.importorskip("oracle")
        pos = clumps(n, [40] * 200, 5)
        mass = np.full(n, 1.0 / n, np.float32)
        args = (torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), 16,
                ((0, 0, 0), 1.0))
        a = tb.build(*args, sorted_keys=True, curve="hilbert")
        b = tb.build(*args, sorted_keys=True, **mode)
        for k in ("perm", "key_sorted", "cell_key", "com", "quad"):
            assert torch.equal(a[k], b[k]), k
        key = a["key_sorted"].cpu().numpy().view(np.uint64)
        perm = a["perm"].cpu().numpy()
        assert np.all((key[1:] > key[:-1]) | ((key[1:] == key[:-1]) & (perm[1:] > perm[:-1])))
    else:
        check(clumps(n, [40] * 200, 5), **mode)
        check((0.25 + 2.0 ** -12 * np.random.default_rng(1).random((n, 3))).astype(np.float32),
              **mode)


@pytest.mark.parametrize("bits", [0, 17])
def test_batch_of_crowded_and_plain_sets(bits):
    """Sets that crowd, sets of coincident points, empty ones and plain ones together."""
    rng = np.random.default_rng(9)
    parts, sizes = [], []
    for k, n in enumerate([5000, 0, 33, 70000, 1, 4096, 100, 20000, 0, 2049]):
        if k % 3 == 0:
            x = 0.5 + 2.0 ** -15 * rng.random((n, 3))
        elif k % 3 == 1:
            x = np.full((n, 3), 0.7)
        else:
            x = rng.random((n, 3))
        parts.append(x.astype(np.float32))
        sizes.append(n)
    for crowd in (True, False):
        if not crowd:  # mostly plain: the sample stays quiet, the runs are sorted one by one
            parts.append(rng.random((900_000, 3), dtype=np.float32)[:900_000])
            sizes.append(900_000)
        pos = np.concatenate(parts)
        if not crowd and bits:
            continue  # the last set is over the bound
        mass = np.full(pos.shape[0], 1.0, np.float32)
        off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
        boxes = np.tile(np.array([0.0, 0.0, 0.0, 1.0]), (len(sizes), 1))
        r = tb.build_batched(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(),
                             torch.from_numpy(off).cuda(), 16, torch.from_numpy(boxes).cuda(),
                             set_index_bits=bits)
        perm = r["perm"].cpu().numpy()
        first = r["cell_first"].cpu().numpy()
        co = r["cell_offsets"].cpu().numpy()
        for b, n in enumerate(sizes):
            if n == 0:
                continue
            ref = oracle.build(pos[off[b]:off[b + 1]], mass[off[b]:off[b + 1]], 16, moments=False)
            assert np.array_equal(perm[off[b]:off[b + 1]] - off[b], ref["perm"]), b
            assert co[b + 1] - co[b] == ref["n_cells"]
            assert np.array_equal(first[co[b]:co[b + 1]] - off[b], ref["cell_first"])

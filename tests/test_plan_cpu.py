"""The host's plan of a build, read from the built library by a small driver
(tests/plan/plan_driver.cpp), against rules restated here.  CPU only."""
import os
import subprocess

import numpy as np
import pytest

import bench
from paper_2312_06102_amd import build_lib
from paper_2312_06102_amd import treebuild as tb

HERE = os.path.dirname(os.path.abspath(__file__))
FORMS = {0: "idx", 2: "key64", 3: "pack64", 4: "pack32"}


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """plans([(n, nsets, n_leaf, flags), ...]) -> a dict of numbers each; with "walk",
    [(n, c_max), ...]."""
    exe = str(tmp_path_factory.mktemp("plan") / "plan_driver")
    lib_dir = os.path.dirname(tb.LIB_PATH)
    cmd = [build_lib.HIPCC, f"--offload-arch={build_lib.ARCH}", "-O1", "-std=c++17", "-x", "hip",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           f"-I{build_lib.INCLUDE}", f"-I{build_lib.CSRC}",
           os.path.join(HERE, "plan", "plan_driver.cpp"), f"-L{lib_dir}", "-ltreebuild",
           f"-Wl,-rpath,{lib_dir}", "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, text=True, timeout=300)

    def ask(rows, *mode):
        text = "\n".join(" ".join(str(int(v)) for v in r) for r in rows)
        r = subprocess.run([exe, *mode], input=text, check=True, capture_output=True, text=True,
                           timeout=300)
        out = []
        for line in r.stdout.splitlines():
            w = line.split()
            out.append({k: int(v) for k, v in zip(w[::2], w[1::2])})
        assert len(out) == len(rows)
        return out
    return ask


def _unfinished(sizes, cell_tile, levels):
    """Whether some set lies over the end of a unit after `levels` rounds of 32 units to
    one: its root has then been built by nobody."""
    tiles = (sizes + cell_tile - 1) // cell_tile
    end = np.cumsum(tiles)
    first, last = (end - tiles)[sizes > 0], (end - 1)[sizes > 0]
    unit = 32 ** levels
    return bool(np.any(first // unit != last // unit))


def test_parents_of_every_set_are_reached(plans):
    """Groups of 32 tiles, then of 32 groups, go on until no set is left over a group's
    end.  Tiles are numbered through all sets, so a small set may lie over any end."""
    rng = np.random.default_rng(31)
    layouts = [[10] * 31 + [1000], [10] * 1023 + [1000, 40], [100] * 1023 + [30_000, 40],
               [500] * 1020 + [400_000, 7], [1] * 16_383, [513], [16_384], [16_385], [600, 5]]
    for _ in range(3000):
        nsets = int(np.exp(rng.uniform(0, np.log(3000))))
        lo = int(np.exp(rng.uniform(np.log(2), np.log(2000))))
        hi = lo * int(rng.choice([2, 16, 128]))
        sizes = np.exp(rng.uniform(np.log(lo), np.log(hi), nsets)).astype(np.int64)
        sizes[rng.random(nsets) < 0.05] = 0
        if sizes.sum() > 0:
            layouts.append(sizes)
    layouts = [np.asarray(s, np.int64) for s in layouts]
    got = plans([(s.sum(), s.size, 16, 0) for s in layouts])
    bad = [(s.size, int(s.sum())) for s, p in zip(layouts, got)
           if _unfinished(s, p["cell_tile"], p["group_levels"])]
    assert not bad, (len(bad), bad[:5])


def test_walk_lists_no_more_items_than_the_workspace_holds(plans):
    """The walk's workspace holds c_max items, and every c_max that bounds the cells is
    accepted: particles in groups (the leaves, say), with c_max from the number of groups
    on."""
    rng = np.random.default_rng(32)
    rows, groups = [], []
    for _ in range(500):
        n = int(np.exp(rng.uniform(0, np.log(10 ** 7))))
        k = max(1, n // int(rng.integers(1, 2000)))
        sizes = np.bincount(rng.integers(0, k, n), minlength=k)
        sizes = sizes[sizes > 0]
        for c_max in {sizes.size, sizes.size + 1, (sizes.size + n) // 2, n, n + 1, 3 * n}:
            if c_max >= sizes.size:
                rows.append((n, c_max))
                groups.append(sizes)
    for (n, c_max), sizes, it in zip(rows, groups, plans(rows, "walk")):
        items = sizes.size if it["whole"] else int(((sizes + it["part"] - 1) // it["part"]).sum())
        assert items <= c_max, (n, c_max, sizes.size, items)
        assert it["part"] <= 1024  # what a workgroup takes in one pass
        if c_max >= n:
            assert not it["whole"]


AUTO_BOX = 0x10000  # the plan's own flag: boxes from the data


@pytest.mark.parametrize("flags", [0, tb.TB_MIXED, tb.TB_SUBTREES, tb.TB_SORT_COUNTED,
                                   tb.TB_SORT_CONFIG(4), tb.TB_SORT_CONFIG(2),
                                   tb.TB_SET_INDEX_BITS(14)])
@pytest.mark.parametrize("nsets", [1, 2, 7, 60, 300, 1000, 16_383])
def test_one_workspace_serves_every_smaller_build(plans, nsets, flags):
    """tb_workspace_bytes never falls as n grows, and no build of n particles needs more
    than it says (with boxes given or from the data)."""
    rng = np.random.default_rng(nsets)
    edges = [2 ** k for k in range(0, 30)] + [3 * 2 ** 18, 2049 * nsets, 32_769 * nsets,
                                              1000 * 1024, 65_536 * 1024]
    sizes = {int(e) + d for e in edges for d in (-2, -1, 0, 1, 2, 4096)}
    sizes |= {int(x) for x in np.exp(rng.uniform(0, np.log(2 ** 29), 400))}
    sizes |= set(range(1, 70)) | set(range(nsets, nsets + 1500, 7))
    sizes = sorted(s for s in sizes if 0 < s <= 2 ** 29)
    for n_leaf in (16, 64, 300):
        said = [tb.tb_workspace_bytes_batched(n, nsets, n_leaf, flags) for n in sizes]
        falls = [(a, b) for a, b, x, y in zip(sizes, sizes[1:], said, said[1:]) if y < x]
        assert not falls, falls[:5]
        for extra in (0, AUTO_BOX):
            need = plans([(n, nsets, n_leaf, flags | extra) for n in sizes])
            for n, x, p in zip(sizes, said, need):
                assert p["total"] <= x, (n, p["total"], x)


def test_what_fits_the_fixed_scratch(plans):
    """tb_build_noalloc goes by the build's own need: just past a size at which the tiles
    grow a build still fits where the largest one before did not."""
    n, n_leaf = 2 ** 20 + 1, 40
    need = plans([(n, 1, n_leaf, AUTO_BOX), (2 ** 20, 1, n_leaf, AUTO_BOX)])
    assert need[0]["total"] < need[1]["total"] <= tb.tb_workspace_bytes(n, n_leaf)


def _forms(p):
    return [FORMS[p[f"form{k}"]] for k in range(p["key_passes"] + 1)]


def _sizes():
    sizes = {1, 2, 3, 2 ** 29 + 12345}
    for b in range(1, 30):
        sizes |= {(1 << b) - 1, 1 << b, (1 << b) + 1}
    return sorted(sizes)


@pytest.mark.parametrize("config,bits", [(0, 8), (2, 8), (4, 9)])
@pytest.mark.parametrize("bound", [0, 5, 18, 28])
def test_large_leaves_sort_every_bit(plans, config, bits, bound):
    """n_leaf above 95: the passes sort all 63 bits and nothing is left to conditional
    passes; at 95 they sort the upper bits."""
    sizes = [n for n in _sizes() if n > 3]
    flags = tb.TB_SORT_CONFIG(config) | tb.TB_SET_INDEX_BITS(bound)
    nsets = 3 if bound else 1
    for n_leaf in (96, 300, 1024):
        for n, p in zip(sizes, plans([(n, nsets, n_leaf, flags) for n in sizes])):
            assert p["bits"] == bits and p["low_passes"] == p["skip_bits"] == 0
            assert _forms(p) == bench.sort_forms(n, bits, bound), n
    for p in plans([(n, nsets, 95, flags) for n in sizes]):
        assert 0 < p["skip_bits"] < 32 and p["low_passes"] >= 2
        assert p["skip_bits"] + p["key_passes"] * bits == 63


@pytest.mark.parametrize("flags", [0, tb.TB_SORT_CONFIG(4)])
@pytest.mark.parametrize("n_leaf", [16, 128])
def test_every_pass_of_every_plan_is_built(plans, n_leaf, flags):
    rows = [(n, nsets, n_leaf, flags | tb.TB_SET_INDEX_BITS(k)) for n in _sizes()
            for nsets in (1, 2, 1000) for k in ((0,) if nsets == 1 else (0, 1, 12, 18, 24, 31))]
    for r, p in zip(rows, plans(rows)):
        assert all(p[f"built{k}"] for k in range(p["key_passes"])), (r, _forms(p))
        # a word holds what is left of the key beside the index
        top = 63 if p["skip_bits"] else 64
        for k in range(1, p["key_passes"]):
            left = top - p["skip_bits"] - k * p["bits"] + p["idx_bits"]
            form = FORMS[p[f"form{k}"]]
            assert left <= {"pack32": 32, "pack64": 64, "key64": 1000}[form], (r, k, form)


@pytest.mark.parametrize("config,bits", [(0, 8), (4, 9)])
@pytest.mark.parametrize("bound", [0, 12, 18, 31])
def test_byte_model_of_the_upper_bits(plans, config, bits, bound):
    """bench.upper_sort_bytes adds up the formats of the plan."""
    rows = [(n, 5 if bound else 1, 16, tb.TB_SORT_CONFIG(config) | tb.TB_SET_INDEX_BITS(bound))
            for n in _sizes()]
    size = {"key64": 8, "pack64": 8, "pack32": 4, "idx": 4}
    for (n, *_), p in zip(rows, plans(rows)):
        f = _forms(p)
        want = n * sum(size[a] + size[b] for a, b in zip(f, f[1:]))
        assert bench.upper_sort_bytes(n, bits, p["key_passes"], bound) == want, (n, f)


def _emulate(keys, p):
    """The passes of a plan as the kernels compute them: the first reads whole keys and drops
    what is not sorted (and the leading 1, unless every bit is); a packed word has its digit
    at bit idx_bits.  Every pass's digit is the key's (as the key kernel counts it)."""
    bits, ib, skip = p["bits"], p["idx_bits"], p["skip_bits"]
    u = np.uint64
    words, idx = keys.copy(), np.arange(keys.shape[0], dtype=np.uint64)
    for k in range(p["key_passes"]):
        fi, fo = FORMS[p[f"form{k}"]], FORMS[p[f"form{k + 1}"]]
        shift = skip + k * bits if fi == "key64" else ib
        if fi != "key64":
            idx = words & u((1 << ib) - 1)
        elif fo != "key64" and skip > 0:
            words = words & u((1 << 63) - 1)
        d = (words >> u(shift)) & u((1 << bits) - 1)
        want = (keys[idx.astype(np.int64)] >> u(skip + k * bits)) & u((1 << bits) - 1)
        assert np.array_equal(d, want), (k, fi)
        order = np.argsort(d, kind="stable")
        words, idx = words[order], idx[order]
        if fo in ("pack64", "pack32"):
            words = ((words >> u(shift + bits)) << u(ib)) | idx
            if fo == "pack32":
                assert not np.any(words >> u(32))
    return idx


@pytest.mark.parametrize("config", [0, 4])
@pytest.mark.parametrize("n_leaf", [16, 128])
@pytest.mark.parametrize("log_n", [1, 2, 7, 12, 16, 17, 18, 19, 23, 24, 25, 26, 28])
def test_passes_sort_stably_by_the_bits_of_the_plan(plans, config, n_leaf, log_n):
    p = plans([(1 << log_n, 1, n_leaf, tb.TB_SORT_CONFIG(config))])[0]
    rng = np.random.default_rng(log_n * 10 + config)
    n = min(4000, 1 << log_n)
    body = rng.integers(0, 1 << 63, n, dtype=np.uint64)
    # duplicates, keys that differ only in the lowest or highest bits, or below the sorted ones
    body[::7] = body[1::7][: body[::7].shape[0]]
    body[3::11] ^= np.uint64(1)
    body[5::13] ^= np.uint64(1 << 62)
    body[2::5] = (body[2::5] & np.uint64(2 ** 20 - 1)) | np.uint64(5 << 40)
    keys = body | np.uint64(1 << 63)
    got = _emulate(keys, p)
    assert np.array_equal(got, np.argsort(keys >> np.uint64(p["skip_bits"]), kind="stable"))


@pytest.mark.parametrize("log_n", [10, 17, 18, 19, 24, 25, 28])
@pytest.mark.parametrize("config", [0, 4])
def test_conditional_passes_meet_the_upper_ones(plans, config, log_n):
    """The digits of the conditional passes cover the bits that the others leave, and their
    packed output, where the plan has it, fits one word."""
    for n in (1 << log_n, (1 << log_n) + 1):
        p = plans([(n, 1, 16, tb.TB_SORT_CONFIG(config))])[0]
        low = [max(0, p["skip_bits"] - p["bits"] * (p["low_passes"] - k))
               for k in range(p["low_passes"])]
        assert low == [p[f"low{k}"] for k in range(p["low_passes"])]
        assert low[0] == 0 and all(b <= a + p["bits"] for a, b in zip(low, low[1:]))
        assert low[-1] + p["bits"] == p["skip_bits"]
        assert p["low_packed"] == (63 - p["skip_bits"] + p["idx_bits"] <= 64)

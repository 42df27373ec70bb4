"""The calls that programs on this framework spend their time in, as measurable cases.

Every case goes through the public entry points of ``treebuild`` and ``simulate``: a kept
``Builder`` or ``BatchBuilder`` launched again on new particles, the one-shot ``build``, a
replayed graph, the walk over a fresh tree, and whole leapfrog steps.  Inputs are drawn on the
GPU from the distributions the benchmark uses (uniform, Plummer, exponential disk, clustered
halos; equal or log-normal masses).  ``exact`` restates the method in plain 64-bit torch.

``TB_SUBTREES`` is not among the cases: it gives the default path's tree more slowly and exists
to show the paper's decomposition, so no program selects it for its work.
"""
import math

import numpy as np
import torch

from paper_2312_06102_amd import simulate
from paper_2312_06102_amd import treebuild as tb

LEVELS = tb.TB_MAX_DEPTH + 1
UNIT_BOX = ((0.0, 0.0, 0.0), 1.0)
EPS = 5e-4  # softening of the walks, as in the benchmark's runs


# ----------------------------------------------------------------------------
# the cases
# ----------------------------------------------------------------------------

def _build(name, dist, n, n_leaf=16, **kw):
    c = dict(name=name, kind="build", dist=dist, n=n, n_leaf=n_leaf, masses="equal",
             precision="fp64", curve="morton", auto_box=False, sorted=False, keys=False)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest tree that is worth one: latency and launch count are all there is
        _build("build_1k", "uniform", 1000, auto_box=True),
        # the benchmark's small workload: everything fits in L2
        _build("build_64k", "uniform", 65536),
        # a script that builds one tree and reads it: allocation, build and read-back
        dict(name="oneshot_300k", kind="oneshot", dist="disk", n=300_007, n_leaf=16,
             masses="lognormal", precision="fp64", curve="morton", auto_box=True),
        # the tree of one time step of a run: box from the data, particles wanted in key order
        _build("build_2m", "plummer", 2_000_003, 10, auto_box=True, sorted=True, keys=True),
        # the headline benchmark
        _build("build_16m", "plummer", 1 << 24),
        # the benchmark's mixed-precision workload
        _build("build_16m_mixed", "clustered", 1 << 24, 8, masses="lognormal",
               precision="mixed"),
        # the largest single set of the benchmark: cosmology-like, small leaves
        _build("build_64m", "clustered", 1 << 26, 8),
        # the benchmark's batch (log-uniform set sizes) at a quarter of its sets
        dict(name="batch_1024", kind="batch", nsets=1024, lo=256, hi=262144, n_leaf=16,
             precision="fp64", curve="morton", auto_box=False, bound=True, graph=False),
        # many little systems, one graph replayed: ragged sets smaller than a tile or two
        dict(name="batch_small", kind="batch", nsets=300, lo=100, hi=4000, n_leaf=16,
             precision="fp64", curve="morton", auto_box=True, bound=False, graph=True),
        # forces on a snapshot: a Peano-Hilbert tree and its walk
        dict(name="forces_300k", kind="forces", dist="disk", n=300_007, n_leaf=16,
             masses="lognormal", curve="hilbert", theta=0.75, n_crit=512, quadrupole=True),
        # a small run stepping: launches of every phase, few groups for the walk
        dict(name="sim_16k", kind="sim", dist="plummer", n=16384, n_leaf=10, theta=0.75,
             n_crit=512, quadrupole=True, reorder_every=1),
        # the benchmark's run at half its size
        dict(name="sim_2m", kind="sim", dist="plummer", n=1 << 21, n_leaf=10, theta=0.75,
             n_crit=512, quadrupole=True, reorder_every=10),
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["build", "build", "build", "oneshot", "batch", "forces", "sim"])
    dist = rng.choice(["uniform", "plummer", "disk", "clustered"])
    n_leaf = rng.choice([8, 10, 16, 16, 32])
    masses = rng.choice(["equal", "lognormal"])
    if kind == "build":
        return dict(kind="build", dist=dist, n=_log_int(rng, 300, 1 << 25), n_leaf=n_leaf,
                    masses=masses, precision=rng.choice(["fp64", "fp64", "mixed"]),
                    curve=rng.choice(["morton", "morton", "morton", "hilbert"]),
                    auto_box=rng.random() < 0.5, sorted=rng.random() < 0.5,
                    keys=rng.random() < 0.3)
    if kind == "oneshot":
        return dict(kind="oneshot", dist=dist, n=_log_int(rng, 300, 1 << 22), n_leaf=n_leaf,
                    masses=masses, precision=rng.choice(["fp64", "mixed"]), curve="morton",
                    auto_box=rng.random() < 0.5)
    if kind == "batch":
        lo = _log_int(rng, 50, 2000)
        hi = lo * rng.choice([2, 16, 128])
        return dict(kind="batch", nsets=_log_int(rng, 2, 1000), lo=lo, hi=hi, n_leaf=n_leaf,
                    precision=rng.choice(["fp64", "fp64", "mixed"]),
                    curve=rng.choice(["morton", "morton", "hilbert"]),
                    auto_box=rng.random() < 0.5, bound=rng.random() < 0.5,
                    graph=rng.random() < 0.5)
    theta, n_crit = rng.choice([0.5, 0.75, 0.75, 1.0]), rng.choice([64, 256, 512, 512])
    quadrupole = rng.random() < 0.75
    if kind == "forces":
        return dict(kind="forces", dist=dist, n=_log_int(rng, 1000, 400_000), n_leaf=n_leaf,
                    masses=masses, curve=rng.choice(["morton", "morton", "hilbert"]),
                    theta=theta, n_crit=n_crit, quadrupole=quadrupole)
    return dict(kind="sim", dist="plummer", n=_log_int(rng, 1000, 400_000), n_leaf=n_leaf,
                theta=theta, n_crit=n_crit, quadrupole=quadrupole,
                reorder_every=rng.choice([1, 10]))


# ----------------------------------------------------------------------------
# particles
# ----------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float64)


def _isotropic(g, n):
    v = torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64)
    return v / v.norm(dim=1, keepdim=True).clamp_min(1e-300)


def _unit_cube(x):
    """The point cloud centred in the unit cube, in FP32, and the length scale."""
    mn, mx = x.amin(0), x.amax(0)
    s = float((mx - mn).max()) * (1.0 + 2.0 ** -20) or 1.0
    y = (0.5 + (x - 0.5 * (mn + mx)) / s).float()
    return y.clamp_(0.0, 1.0 - 2.0 ** -24), s


def _plummer_radii(g, n, rmax=50.0):
    u = _rand(g, n) * (rmax ** 3 * (1.0 + rmax ** 2) ** -1.5)
    return (u.clamp_min(1e-300) ** (-2.0 / 3.0) - 1.0) ** -0.5


def _bisect(f, target, hi, steps=44):
    lo = torch.zeros_like(target)
    hi = torch.zeros_like(target) + hi
    for _ in range(steps):
        mid = 0.5 * (lo + hi)
        below = f(mid) < target
        lo = torch.where(below, mid, lo)
        hi = torch.where(below, hi, mid)
    return 0.5 * (lo + hi)


def _disk(g, n):
    """Exponential disk (scale length 1, sech^2 height 0.1, truncated at 10)."""
    def frac(r):
        return 1.0 - (1.0 + r) * torch.exp(-r)
    r = _bisect(frac, _rand(g, n) * (1.0 - 11.0 * math.exp(-10.0)), 10.0)
    phi = _rand(g, n) * (2.0 * math.pi)
    z = 0.1 * torch.atanh((2.0 * _rand(g, n) - 1.0).clamp(-1.0 + 1e-15, 1.0 - 1e-15))
    return torch.stack([r * torch.cos(phi), r * torch.sin(phi), z], 1)


def _clustered(g, n, seed):
    """70 % of the particles in NFW halos with dN/dM ~ M^-1.9, the rest uniform."""
    rng = np.random.default_rng(int(seed))
    n_h = int(round(0.7 * n))
    halos = max(1, min(2000, n_h // 20))
    a = 1.0 - 1.9
    m = (1e2 ** a + rng.random(halos) * (1e6 ** a - 1e2 ** a)) ** (1.0 / a)
    counts = np.floor(m * (n_h / m.sum())).astype(np.int64)
    counts[0] += n_h - counts.sum()
    counts = torch.from_numpy(counts).cuda()
    conc = torch.from_numpy(rng.uniform(5.0, 15.0, halos)).cuda()
    centre = torch.from_numpy(rng.random((halos, 3))).cuda()
    r200 = (3.0 * counts.double() / (4.0 * math.pi * 200.0 * n)) ** (1.0 / 3.0)

    def mu(x):
        return torch.log1p(x) - x / (1.0 + x)
    c = conc.repeat_interleave(counts)
    r = _bisect(mu, _rand(g, n_h) * mu(c), c, 40) * (r200 / conc).repeat_interleave(counts)
    x = centre.repeat_interleave(counts, 0) + r[:, None] * _isotropic(g, n_h)
    x = torch.cat([x, _rand(g, n - n_h, 3)]).remainder(1.0).float()
    x[x >= 1.0] = 0.0
    return x[torch.randperm(n, generator=g, device="cuda")]


def _positions(dist, n, seed):
    g = _gen(seed)
    if dist == "uniform":
        return torch.rand(n, 3, generator=g, device="cuda")
    if dist == "plummer":
        return _unit_cube(_plummer_radii(g, n)[:, None] * _isotropic(g, n))[0].contiguous()
    if dist == "disk":
        return _unit_cube(_disk(g, n))[0].contiguous()
    return _clustered(g, n, seed).contiguous()


def _masses(kind, n, seed):
    if kind == "equal":
        return torch.full((n,), 1.0 / n, device="cuda", dtype=torch.float32)
    m = torch.exp(torch.randn(n, generator=_gen(seed + 77), device="cuda", dtype=torch.float64))
    return (m / m.sum()).float().clamp_min(torch.finfo(torch.float32).tiny)


def _particles(case, seed):
    mass = _masses(case.get("masses", "equal"), case["n"], seed)
    if case["kind"] == "oneshot":
        # a one-shot build returns as many cells as there are: the seed gives the order and
        # the masses, the case the positions, so that every seed has the same number
        order = torch.randperm(case["n"], generator=_gen(seed), device="cuda")
        return _positions(case["dist"], case["n"], 7)[order], mass
    return _positions(case["dist"], case["n"], seed), mass


def _sim_particles(case, seed):
    """A Plummer sphere in equilibrium, G = 1, total mass 1, in the unit cube."""
    g, n = _gen(seed), case["n"]
    r = _plummer_radii(g, n)
    x = r[:, None] * _isotropic(g, n)
    q = torch.zeros(n, device="cuda", dtype=torch.float64)
    todo = torch.arange(n, device="cuda")
    while todo.numel():  # speeds by rejection (Aarseth, Henon & Wielen 1974)
        x1, x2 = _rand(g, todo.numel()), _rand(g, todo.numel())
        ok = 0.1 * x2 < x1 * x1 * (1.0 - x1 * x1) ** 3.5
        q[todo[ok]] = x1[ok]
        todo = todo[~ok]
    v = (q * math.sqrt(2.0) * (1.0 + r * r) ** -0.25)[:, None] * _isotropic(g, n)
    pos, s = _unit_cube(x)
    return pos.contiguous(), (v * math.sqrt(s)).float(), _masses("equal", n, seed)


def _set_sizes(case):
    """The sizes belong to the case, so that every seed of it is the same amount of work."""
    rng = np.random.default_rng(case["nsets"] * 1_000_003 + case["lo"] * 101 + case["hi"])
    u = rng.uniform(math.log(case["lo"]), math.log(case["hi"]), case["nsets"])
    return np.floor(np.exp(u)).astype(np.int64)


def _batch_particles(case, seed):
    """Independent Plummer spheres, each scaled into its own unit cube, masses 1/n_b."""
    sizes = torch.from_numpy(_set_sizes(case)).cuda()
    off = torch.zeros(case["nsets"] + 1, dtype=torch.int64, device="cuda")
    off[1:] = sizes.cumsum(0)
    n = int(off[-1])
    g = _gen(seed)
    x = _plummer_radii(g, n)[:, None] * _isotropic(g, n)
    b = torch.arange(case["nsets"], device="cuda").repeat_interleave(sizes)
    idx = b[:, None].expand(-1, 3)
    shape = (case["nsets"], 3)
    mn = torch.full(shape, math.inf, device="cuda", dtype=torch.float64)
    mn = mn.scatter_reduce(0, idx, x, "amin")
    mx = torch.full(shape, -math.inf, device="cuda", dtype=torch.float64)
    mx = mx.scatter_reduce(0, idx, x, "amax")
    s = (mx - mn).amax(1) * (1.0 + 2.0 ** -20)
    y = 0.5 + (x - (0.5 * (mn + mx))[b]) / s[b, None]
    pos = y.float().clamp_(0.0, 1.0 - 2.0 ** -24).contiguous()
    return pos, (1.0 / sizes.double())[b].float().contiguous(), off


def _boxes(case):
    if case["auto_box"]:
        return None
    return torch.tensor([[0.0, 0.0, 0.0, 1.0]], device="cuda",
                        dtype=torch.float64).repeat(case["nsets"], 1)


# ----------------------------------------------------------------------------
# what a program holds, and one pass
# ----------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind == "sim":
        pos, vel, mass = (t.cpu().numpy() for t in _sim_particles(case, seed))
        sim = simulate.Simulation(pos, vel, mass, 1e-4, n_leaf=case["n_leaf"],
                                  theta=case["theta"], n_crit=case["n_crit"], eps=EPS,
                                  reorder_every=case["reorder_every"],
                                  quadrupole=case["quadrupole"])
        sim.step(1)  # a run under way: forces known, velocities half a step behind
        return dict(kind=kind, sim=sim)
    if kind == "batch":
        pos, mass, off = _batch_particles(case, seed)
        bits = max(1, int(_set_sizes(case).max() - 1).bit_length()) if case["bound"] else 0
        b = tb.BatchBuilder(pos.shape[0], case["nsets"], case["n_leaf"], case["precision"],
                            curve=case["curve"], set_index_bits=bits)
        args = (pos, mass, off, _boxes(case))
        outputs = dict(_outputs(b), cell_offsets=b.cell_offsets)
        if case["graph"]:
            b.capture(*args)
        return dict(kind=kind, b=b, args=args, outputs=outputs, graph=case["graph"])
    pos, mass = _particles(case, seed)
    if kind == "oneshot":
        return dict(kind=kind, pos=pos, mass=mass, n_leaf=case["n_leaf"],
                    box=None if case["auto_box"] else UNIT_BOX, precision=case["precision"])
    if kind == "forces":
        b = tb.Builder(case["n"], case["n_leaf"], sorted_particles=True, curve=case["curve"])
        return dict(kind=kind, b=b, pos=pos, mass=mass, theta=case["theta"],
                    n_crit=case["n_crit"], quadrupole=case["quadrupole"])
    b = tb.Builder(case["n"], case["n_leaf"], case["precision"], sorted_particles=case["sorted"],
                   sorted_keys=case["keys"], curve=case["curve"])
    return dict(kind=kind, b=b, pos=pos, mass=mass, outputs=_outputs(b),
                box=None if case["auto_box"] else UNIT_BOX)


def _outputs(builder):
    """The builder's output buffers.  They hold C_max cells; those past the tree's last one
    are never written and read as zero here."""
    out = {k: v for k, v in vars(builder.out).items() if v is not None}
    for v in out.values():
        v.zero_()
    return out


def run(state):
    kind = state["kind"]
    if kind == "build":
        state["b"].launch(state["pos"], state["mass"], state["box"])
        return state["outputs"]
    if kind == "batch":
        if state["graph"]:
            state["b"].replay()
        else:
            state["b"].launch(*state["args"])
        return state["outputs"]
    if kind == "oneshot":
        return tb.build(state["pos"], state["mass"], state["n_leaf"], state["box"],
                        state["precision"])
    if kind == "forces":
        b = state["b"]
        b.launch(state["pos"], state["mass"], UNIT_BOX)
        acc, stats = b.gravity(state["theta"], state["n_crit"], EPS, state["quadrupole"])
        return dict(acc=acc, groups=stats["groups"], interactions=stats["interactions"],
                    perm=b.out.perm)
    sim = state["sim"]
    sim.step(1)
    return dict(pos=sim.pos, vel=sim.vel, mass=sim.mass, ids=sim.ids, acc=sim.acc)


def _n(case):
    return int(_set_sizes(case).sum()) if case["kind"] == "batch" else case["n"]


def work(case):
    n = _n(case)
    cells = 3.7 * n / case["n_leaf"] + 8  # what these distributions come to
    wide = 4 if case.get("precision") == "mixed" else 8
    # positions and masses in; perm and the cells (key, level, first, count, children, com,
    # quadrupole) out
    nbytes = n * (16 + 4) + cells * (8 + 1 + 4 + 4 + 8 + 10 * wide)
    flops = 45.0 * n + 60.0 * cells  # moments of the leaves, then of their parents
    if case.get("sorted"):
        nbytes += 16 * n
    if case.get("keys"):
        nbytes += 8 * n
    if case["kind"] in ("forces", "sim"):
        listed_ = _list_length(case)
        nbytes += n * 32 + (n * 24 * 2 if case["kind"] == "sim" else 0)
        flops += n * listed_ * (60.0 if case["quadrupole"] else 25.0)
    return {"bytes": nbytes, "flops": flops}


def _list_length(case):
    """Interactions a particle has: about, for the walk's settings."""
    grow = max(1.0, math.log2(case["n"] / case["n_crit"]))
    return min(case["n"], 1.4 * case["n_crit"] + 75.0 * grow / case["theta"] ** 2)


# ----------------------------------------------------------------------------
# the same results in plain 64-bit torch
# ----------------------------------------------------------------------------

def _spread(v):
    out = torch.zeros_like(v)
    for b in range(21):
        out |= ((v >> b) & 1) << (3 * b)
    return out


def _hilbert(q):
    """Skilling's transpose of 21-bit coordinates (AIP Conf. Proc. 707, 381, 2004)."""
    x = [q[:, 0].clone(), q[:, 1].clone(), q[:, 2].clone()]
    bit = 1 << 20
    while bit > 1:
        low = bit - 1
        for a in range(3):
            on = (x[a] & bit) != 0
            t = torch.where(on, torch.zeros_like(x[0]), (x[0] ^ x[a]) & low)
            x[0] = torch.where(on, x[0] ^ low, x[0] ^ t)
            if a:
                x[a] = x[a] ^ t
        bit >>= 1
    x[1] = x[1] ^ x[0]
    x[2] = x[2] ^ x[1]
    t = torch.zeros_like(x[0])
    bit = 1 << 20
    while bit > 1:
        t = torch.where((x[2] & bit) != 0, t ^ (bit - 1), t)
        bit >>= 1
    return torch.stack([x[0] ^ t, x[1] ^ t, x[2] ^ t], 1)


def _seg_sum(v, start, count):
    """Sums of the consecutive runs [start, start + count) that cover v."""
    if count.numel() <= 64:
        at = start.tolist()
        return torch.stack([v[a:a + c].sum() for a, c in zip(at, count.tolist())])
    return torch.segment_reduce(v, "sum", lengths=count, unsafe=True)


def _auto_boxes(pos, off):
    out = []
    for b in range(off.numel() - 1):
        x = pos[int(off[b]):int(off[b + 1])].double()
        mn = x.amin(0)
        ext = float((x.amax(0) - mn).max())
        out.append(mn.tolist() + [math.ldexp(1.0, math.frexp(ext)[1]) if ext > 0 else 1.0])
    return torch.tensor(out, device="cuda", dtype=torch.float64)


def _tree64(pos, mass, off, boxes, n_leaf, curve, links=False):
    """The trees of the sets [off[b], off[b+1]), cells in (set, depth, key) order."""
    n, nsets = pos.shape[0], off.numel() - 1
    sid = torch.arange(nsets, device="cuda").repeat_interleave(off[1:] - off[:-1])
    x = pos.double() - boxes[sid, :3]
    q = torch.floor(x * (2097152.0 / boxes[sid, 3])[:, None]).clamp(0, 2097151).long()
    k = _hilbert(q) if curve == "hilbert" else q
    key = (_spread(k[:, 0]) << 2) | (_spread(k[:, 1]) << 1) | _spread(k[:, 2])
    del k
    perm = torch.sort(key, stable=True)[1]
    if nsets > 1:
        perm = perm[torch.sort(sid[perm], stable=True)[1]]
    key, q, x, m, sid = key[perm], q[perm], x[perm], mass.double()[perm], sid[perm]
    parts, act, par, base = [], torch.arange(n, device="cuda"), None, 0
    for d in range(LEVELS):
        pre, s = key[act] >> (63 - 3 * d), sid[act]
        new = torch.ones(act.numel(), dtype=torch.bool, device="cuda")
        new[1:] = (pre[1:] != pre[:-1]) | (s[1:] != s[:-1])
        start = new.nonzero().flatten()
        count = torch.diff(start, append=torch.tensor([act.numel()], device="cuda"))
        cid = new.cumsum(0) - 1
        first = act[start]
        side = boxes[s[start], 3] * 2.0 ** -d
        cen = ((q[first] >> (21 - d)).double() + 0.5) * side[:, None]
        ma = m[act]
        big = _seg_sum(ma, start, count)
        r = x[act] - cen[cid]
        com = torch.stack([_seg_sum(ma * r[:, a], start, count) / big for a in range(3)], 1)
        r -= com[cid]
        w = ma * (r * r).sum(1)
        quad = []
        for a, b in ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2)):
            t = 3.0 * ma * r[:, a] * r[:, b]
            quad.append(_seg_sum(t - w if a == b else t, start, count))
        p = dict(com=torch.cat([com, big[:, None]], 1), quad=torch.stack(quad, 1),
                 set=s[start])
        if links:
            p.update(depth=torch.full_like(first, d), first=first, count=count, centre=cen,
                     side=side, parent=par[start] if par is not None else first * 0 - 1,
                     leaf=(count <= n_leaf) if d < 21 else count > 0)
        parts.append(p)
        keep = (count > n_leaf)[cid] if d < 21 else cid < 0
        par = cid[keep] + base
        base += first.numel()
        act = act[keep]
        if not act.numel():
            break
    tree = {f: torch.cat([p[f] for p in parts]) for f in parts[0]}
    if nsets > 1:
        o = torch.sort(tree["set"], stable=True)[1]
        tree = {f: v[o] for f, v in tree.items()}
    tree["perm"], tree["x"], tree["m"] = perm, x, m
    return tree


def _ranges(first, count):
    """The positions of every run, one after the other, and the run of each."""
    run_ = torch.arange(first.numel(), device="cuda").repeat_interleave(count)
    ends = count.cumsum(0)
    return first[run_] + torch.arange(run_.numel(), device="cuda") - (ends - count)[run_], run_


def _walk64(t, n, theta, n_crit, quadrupole):
    """Accelerations and potentials in key order by the group walk over tree t."""
    par, cnt, leaf = t["parent"], t["count"], t["leaf"]
    small = (cnt <= n_crit) | leaf
    up = par.clamp_min(0)
    grp = (small & ((par < 0) | ~small[up])).nonzero().flatten()
    kids = torch.zeros_like(cnt).index_add_(0, par[1:], torch.ones_like(par[1:]))
    kid0 = torch.zeros_like(cnt)
    at = torch.arange(par.numel(), device="cuda")
    kid0.scatter_reduce_(0, par[1:], at[1:], "amin", include_self=False)
    cabs = t["centre"] + t["com"][:, :3]
    acc = torch.zeros(n, 4, device="cuda", dtype=torch.float64)
    g, c = torch.arange(grp.numel(), device="cuda"), torch.zeros_like(grp)
    far, near = [], []
    while g.numel():
        gg = grp[g]
        inside = ((t["depth"][c] <= t["depth"][gg]) & (t["first"][c] <= t["first"][gg])
                  & (t["first"][gg] < t["first"][c] + cnt[c]))
        gap = ((cabs[c] - t["centre"][gg]).abs() - 0.5 * t["side"][gg][:, None]).clamp_min(0)
        take = ~inside & (t["side"][c] ** 2 < theta * theta * (gap * gap).sum(1))
        far.append((gg[take], c[take]))
        opened = ~take & leaf[c]
        near.append((gg[opened], c[opened]))
        g, c = g[~take & ~leaf[c]], c[~take & ~leaf[c]]
        c, src = _ranges(kid0[c], kids[c])
        g = g[src]
    for cells, lists in ((True, far), (False, near)):
        gg, src = (torch.cat(v) for v in zip(*lists))
        if not cells:
            src, of = _ranges(t["first"][src], cnt[src])
            gg = gg[of]
        load = cnt[gg].cumsum(0)
        a, total = 0, gg.numel()
        while a < total:
            done = int(load[a - 1]) if a else 0
            b = max(a + 1, int(torch.searchsorted(load, done + 16_000_000, right=True)))
            i, of = _ranges(t["first"][gg[a:b]], cnt[gg[a:b]])
            s = src[a:b][of]
            if cells:
                _add_cells(acc, t, i, s, cabs, quadrupole)
            else:
                i, s = i[i != s], s[i != s]
                r = t["x"][i] - t["x"][s]
                u = (r * r).sum(1).add_(EPS * EPS).rsqrt()
                w = t["m"][s] * u
                acc.index_add_(0, i, torch.cat([-(w * u * u)[:, None] * r, -w[:, None]], 1))
            a = b
    return acc


def _add_cells(acc, t, i, s, cabs, quadrupole):
    r = t["x"][i] - cabs[s]
    u = (r * r).sum(1).rsqrt()
    mass = t["com"][s, 3]
    v = -(mass * u ** 3)[:, None] * r
    phi = -mass * u
    if quadrupole:
        q = t["quad"][s]
        qr = torch.stack([q[:, 0] * r[:, 0] + q[:, 1] * r[:, 1] + q[:, 2] * r[:, 2],
                          q[:, 1] * r[:, 0] + q[:, 3] * r[:, 1] + q[:, 4] * r[:, 2],
                          q[:, 2] * r[:, 0] + q[:, 4] * r[:, 1] + q[:, 5] * r[:, 2]], 1)
        rqr = (qr * r).sum(1)
        v += (u ** 5)[:, None] * qr - (2.5 * rqr * u ** 7)[:, None] * r
        phi = phi - 0.5 * rqr * u ** 5
    acc.index_add_(0, i, torch.cat([v, phi[:, None]], 1))


def _padded(v, case):
    """v with rows of zeros up to the C_max cells of the builder's buffers."""
    n = _n(case)
    rows = n + 21 * (n // (case["n_leaf"] + 1))
    return torch.cat([v, v.new_zeros(rows - v.shape[0], v.shape[1])])


def _whole(n):
    return torch.tensor([0, n], device="cuda")


def exact(case, seed):
    kind = case["kind"]
    if kind == "sim":
        return _exact_sim(case, seed)
    if kind == "batch":
        pos, mass, off = _batch_particles(case, seed)
        box = _auto_boxes(pos, off) if case["auto_box"] else _boxes(case)
        t = _tree64(pos, mass, off, box, case["n_leaf"], case["curve"])
        return dict(com=_padded(t["com"], case), quad=_padded(t["quad"], case), box_out=box)
    pos, mass = _particles(case, seed)
    off, unit = _whole(case["n"]), torch.tensor([[0.0, 0.0, 0.0, 1.0]], device="cuda",
                                                dtype=torch.float64)
    if kind == "forces":
        t = _tree64(pos, mass, off, unit, case["n_leaf"], case["curve"], links=True)
        return dict(acc=_walk64(t, case["n"], case["theta"], case["n_crit"],
                                case["quadrupole"]))
    box = _auto_boxes(pos, off) if case["auto_box"] else unit
    t = _tree64(pos, mass, off, box, case["n_leaf"], case["curve"])
    if kind == "oneshot":
        return dict(com=t["com"], quad=t["quad"], box=box[0])
    out = dict(com=_padded(t["com"], case), quad=_padded(t["quad"], case), box_out=box[0])
    if case.get("sorted"):
        out.update(pos_sorted=pos[t["perm"]], mass_sorted=mass[t["perm"]])
    return out


def _exact_sim(case, seed):
    """Two leapfrog steps from the start; positions and velocities are FP32 state."""
    pos, vel, mass = _sim_particles(case, seed)
    n, dt = case["n"], 1e-4
    perm = acc = None
    for step in range(3):
        if step:
            a = torch.empty_like(acc)
            a[perm] = acc
            vel = (vel.double() + a[:, :3] * (dt if step > 1 else 0.5 * dt)).float()
            pos = (pos.double() + vel.double() * dt).float()
        off = _whole(n)
        t = _tree64(pos, mass, off, _auto_boxes(pos, off), case["n_leaf"], "morton", links=True)
        acc = _walk64(t, n, case["theta"], case["n_crit"], case["quadrupole"])
        perm = t["perm"]
        if step % case["reorder_every"] == 0:
            pos, vel, mass = pos[perm], vel[perm], mass[perm]
            perm = torch.arange(n, device="cuda")
    return dict(pos=pos, vel=vel, mass=mass, acc=acc)

"""Performance cases of the cluster-pair non-bonded library, each through its public entry points.

A case is a dict of plain values; `kind` names the call sequence:

  forces   nb_forces on a list that is already built: one MD step between list builds
  cycle    nb_grid_sort + nb_pairlist_build (asynchronous) + nstlist x nb_forces: one list lifetime of MD
  prune    nb_pairlist_prune of a long-lived box-only list + a few nb_forces on the pruned list
  rdf      nb_grid_sort + box-only nb_pairlist_build + nb_rdf: one frame of a pair correlation analysis
  recount  nb_pairlist_build (synchronous) + nb_recount: one label of the learned-buffer data
  batch    nb_batch_replay of a captured cycle (rebuild + nstlist force steps) of many uneven replicas
  mlp      nb_mlp_grad: loss and gradient of one training minibatch of the buffer predictor

The particles are rigid SPC/E waters at liquid density.  To be quick to make at every size they sit on a jittered
lattice, bent by smooth shears, with random vacancies and orientations (O-O distances from about 0.2 nm), and move
ballistically at 300 K with 2 fs steps between list builds.  Units: nm, ps, kJ/mol, e, u.
"""
import math

import numpy as np
import torch

import paper_1306_1737_amd as mxn

COULOMB_F = 138.935458
KB = 0.0083144626
MASS_O, MASS_H = 15.9994, 1.008
Q_O, Q_H = -0.8476, 0.4238
C6 = 4.0 * 0.650 * 0.3166 ** 6
C12 = 4.0 * 0.650 * 0.3166 ** 12
PER_NM3 = 602.214076 / (MASS_O + 2.0 * MASS_H)   # waters per nm^3 at 1 g/cm^3
DT = 0.002
MLP_LO = [280.0, 0.0, 5.0, 0.95, 0.8, 0.0, 0.0, 0.0]
MLP_HI = [360.0, 0.25, 40.0, 1.05, 1.2, 1.0, 1.0, 1.0]
RECOUNT_DB, RECOUNT_SPAN = 0.002, 0.5


def _beta(rc):
    return 3.1234132 / rc   # erfc(beta rc) = 1e-5


def _md(name, kind, waters, shape, rc, rlist, **more):
    m, n = (int(v) for v in shape.split("x"))
    case = {"kind": kind, "waters": waters, "m": m, "n": n, "rc": rc, "rlist": rlist, "aspect": 1.0, "nstlist": 10,
            "energy": True, "virial": False, "coulomb": "ewald"}
    case.update(more)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest systems: a few hundred molecules, where launches and latency are all there is
        _md("forces_900_8x8", "forces", 300, "8x8", 0.9, 1.0),
        # a small box at the paper's 4x4 CPU shape through one list lifetime
        _md("cycle_3k_4x4", "cycle", 1000, "4x4", 0.9, 1.0),
        # a peptide-sized slab at the paper's GPU shape; plain force steps, no energies
        _md("cycle_12k_8x4", "cycle", 4001, "8x4", 1.0, 1.1, aspect=1.5, nstlist=20, energy=False),
        # mid-sized box at the third shape, reaction field with a conducting boundary
        _md("forces_24k_4x8_rf", "forces", 7919, "4x8", 1.0, 1.1, coulomb="rf"),
        # the production box: list lifetime of ten steps with energies
        _md("cycle_96k_8x8", "cycle", 32000, "8x8", 1.0, 1.1),
        # a pressure-coupled step of the production box: energies and virial
        _md("forces_96k_8x8_virial", "forces", 32000, "8x8", 1.0, 1.1, virial=True),
        # the rolling two-stage schedule: one prune and the four steps it lasts
        _md("prune_96k_8x8", "prune", 32000, "8x8", 1.0, 1.3, nstlist=4),
        # trajectory analysis: every frame sorted, listed and histogrammed
        _md("rdf_96k_8x8", "rdf", 32000, "8x8", 1.0, 1.01),
        # training data of the learned buffer: synchronous list and exact recount
        _md("recount_12k_4x4", "recount", 4000, "4x4", 1.0, 1.5),
        # many uneven replicas of 1 500 to 24 000 atoms, one captured cycle per replay
        _md("batch_64_8x4", "batch", 500, "8x4", 1.0, 1.1, replicas=64, largest=8000),
        # one minibatch of the buffer predictor's training
        {"name": "mlp_256", "kind": "mlp", "batch": 256},
        # the largest box: three million atoms, sorted, listed and evaluated once with energies and virial
        _md("cycle_3M_8x8", "cycle", 1000000, "8x8", 1.0, 1.1, nstlist=1, virial=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forces", "forces", "cycle", "cycle", "cycle", "prune", "rdf", "recount", "batch", "mlp"])
    if kind == "mlp":
        return {"kind": "mlp", "batch": _log(rng, 32, 2048)}
    shape = rng.choice(["4x4", "4x8", "8x4", "8x8", "8x8"])
    if kind == "batch":
        lo = _log(rng, 400, 2000)
        return _md(None, kind, lo, shape, 1.0, 1.1, replicas=_log(rng, 4, 64), largest=lo + _log(rng, 400, 6000),
                   nstlist=rng.randint(5, 10), coulomb=rng.choice(["ewald", "rf", "table"]))
    aspect = rng.choice([1.0, round(rng.uniform(1.0, 2.0), 2)])
    if kind == "recount":
        rc = round(rng.uniform(0.8, 1.2), 3)
        return _md(None, kind, _log(rng, 2500, 8000), rng.choice(["4x4", "4x8", "8x8"]), rc, rc + RECOUNT_SPAN)
    lo, hi = {"forces": (300, 200000), "cycle": (300, 50000), "rdf": (300, 60000), "prune": (1500, 60000)}[kind]
    waters = _log(rng, lo, hi)
    half = 0.49 * (waters / PER_NM3 / aspect) ** (1.0 / 3.0)   # half the shortest edge
    rc = round(min(rng.uniform(0.8, 1.2), half - 0.16), 3)
    if kind == "rdf":
        return _md(None, kind, waters, shape, rc, rc + 0.01, aspect=aspect)
    if kind == "prune":
        rc = min(rc, round(half - 0.31, 3))
        return _md(None, kind, waters, shape, rc, rc + 0.3, aspect=aspect, nstlist=rng.randint(3, 6))
    virial = waters >= 20000 and rng.random() < 0.5   # pressure-coupled steps: boxes of production size
    energy = virial or rng.random() < 0.6
    return _md(None, kind, waters, shape, rc, round(rc + rng.uniform(0.05, 0.15), 3), aspect=aspect,
               nstlist=rng.randint(5, 20) if kind == "cycle" else 10, energy=energy, virial=virial,
               coulomb=rng.choice(["ewald", "ewald", "rf", "table"]))


# ------------------------------------------------------------------- inputs

def _box(waters, aspect):
    edge = (waters / PER_NM3 / aspect) ** (1.0 / 3.0)
    return np.array([edge, edge, edge * aspect])


def _water(rng, waters, box):
    """(3 waters, 3) float32 positions (O, H, H per molecule) and the (3 waters, 3) velocities at 300 K."""
    a = (box.prod() / waters) ** (1.0 / 3.0)
    sites = np.maximum(1, np.rint(box / a)).astype(np.int64)
    while sites.prod() < waters:
        sites[np.argmax(box / sites)] += 1
    pick = rng.permutation(int(sites.prod()))[:waters]
    cell = np.stack(np.unravel_index(pick, sites), axis=1)
    o = (cell + 0.5 + rng.uniform(-0.1, 0.1, (waters, 3))) * (box / sites)
    # gentle periodic shears (each keeps the density) bend the lattice rows, so that no grid is aligned with them
    for d, (p, q) in enumerate(((1, 2), (2, 0), (0, 1))):
        waves = np.sin(2.0 * np.pi * (o[:, (p, q)] / box[[p, q]] + rng.uniform(0.0, 1.0, 2))).sum(1)
        o[:, d] += 0.45 * box[d] / sites[d] * waves
    u = rng.standard_normal((waters, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    w = rng.standard_normal((waters, 3))
    w -= (w * u).sum(1, keepdims=True) * u
    w /= np.linalg.norm(w, axis=1, keepdims=True)
    half = math.radians(109.47) / 2.0
    x = np.stack([o, o + 0.1 * (math.cos(half) * u + math.sin(half) * w),
                  o + 0.1 * (math.cos(half) * u - math.sin(half) * w)], axis=1).reshape(-1, 3)
    mass = np.tile([MASS_O, MASS_H, MASS_H], waters)
    v = rng.standard_normal((3 * waters, 3)) * np.sqrt(KB * 300.0 / mass)[:, None]
    return x.astype(np.float32), v.astype(np.float32)


def _frame(x, v, t, waters):
    """(n, 4) float32: positions after a free flight of t ps, and charges."""
    out = np.empty((3 * waters, 4), np.float32)
    out[:, :3] = x + v * np.float32(t)
    out[:, 3] = np.tile(np.array([Q_O, Q_H, Q_H], np.float32), waters)
    return out


def _steps(case):
    """Free-flight steps at which the case's force calls are made."""
    if case["kind"] == "forces":
        return [5]
    if case["kind"] == "prune":
        return [12 + k for k in range(case["nstlist"])]
    return list(range(case["nstlist"])) if case["kind"] == "cycle" else [0]


def _make_md(case, seed):
    rng = np.random.default_rng([seed, 1306])
    box = _box(case["waters"], case["aspect"])
    x, v = _water(rng, case["waters"], box)
    first = _frame(x, v, 0.0, case["waters"])
    if case["kind"] == "recount":   # free-flight displacement of the list lifetime
        now = [_frame(x, v, (20 - 1) * DT, case["waters"])]
    else:
        now = [_frame(x, v, k * DT, case["waters"]) for k in _steps(case)]
    return box, first, now


def _make_replicas(case, seed):
    rng = np.random.default_rng([seed, 2612])
    sizes = np.rint(np.exp(np.random.default_rng(11).uniform(math.log(case["waters"]), math.log(case["largest"]),
                                                            case["replicas"]))).astype(int)
    reps = []
    for w in sizes:
        box = _box(int(w), 1.0)
        x, v = _water(rng, int(w), box)
        reps.append((int(w), box, _frame(x, v, 0.0, int(w))))
    return reps


def _make_mlp(case, seed):
    rng = np.random.default_rng([seed, 64])
    p = []
    for fan_in, fan_out in ((8, 64), (64, 64)):
        a = math.sqrt(6.0 / (fan_in + fan_out))
        p += [rng.uniform(-a, a, fan_out * fan_in), rng.uniform(-0.1, 0.1, fan_out)]
    a = math.sqrt(6.0 / 65.0)
    p += [rng.uniform(-a, a, 64), [math.log(math.expm1(0.05))]]
    n = case["batch"]
    X = rng.uniform(MLP_LO, MLP_HI, (n, 8))
    X[:, 5:] = np.eye(3)[rng.integers(0, 3, n)]
    X[:, 2] = np.rint(X[:, 2])
    return np.concatenate(p).astype(np.float32), X.astype(np.float32), rng.uniform(0.01, 0.3, n).astype(np.float32)


def _coulomb(case):
    return {"ewald": mxn.NB_COULOMB_EWALD, "rf": mxn.NB_COULOMB_RF, "table": mxn.NB_COULOMB_EWALD_TABLE}[case["coulomb"]]


def _flags(case):
    return (mxn.NB_ENERGY if case["energy"] else 0) | (mxn.NB_VIRIAL if case["virial"] else 0)


class _State:
    """What a program keeps between calls: the context, its handles and its device arrays."""

    def __init__(self, case):
        self.case = case
        self.dev = torch.device("cuda:0")
        self.ctx = mxn.nb_create(0)
        self.grids, self.lists, self.inner, self.batch, self.model = [], [], None, None, None

    def up(self, a):
        return torch.from_numpy(np.ascontiguousarray(a)).to(self.dev)

    def topology(self, waters):
        typ = self.up(np.tile(np.array([0, 1, 1], np.int32), waters))
        base = np.repeat(np.arange(waters) * 3, 3)
        k = np.tile(np.arange(3), waters)
        partners = np.sort(np.stack([base + (k + 1) % 3, base + (k + 2) % 3], axis=1), axis=1)
        return typ, self.up(np.arange(3 * waters + 1, dtype=np.int32) * 2), self.up(partners.reshape(-1).astype(np.int32))

    def params(self):
        c, lj = self.case, np.zeros((2, 2, 2), np.float32)
        lj[0, 0] = C6, C12
        return mxn.make_params(c["rc"], _beta(c["rc"]), COULOMB_F, self.up(lj), coulomb=_coulomb(c))

    def __del__(self):
        if self.batch is not None:
            mxn.nb_batch_free(self.batch)
        if self.model is not None:
            mxn.nb_mlp_free(self.model)
        for lst in self.lists + ([self.inner] if self.inner is not None else []):
            mxn.nb_list_free(lst)
        for g in self.grids:
            mxn.nb_grid_free(g)
        mxn.nb_destroy(self.ctx)


def _rbb(case, box):
    if case["kind"] == "recount":
        spacing = (max(case["m"], case["n"]) / (3 * case["waters"] / box.prod())) ** (1.0 / 3.0)
        return float(np.float32(case["rlist"]) - np.float32(0.5 * spacing)), float(np.float32(0.5 * spacing))
    return (case["rlist"], 0.0) if case["kind"] in ("prune", "rdf") else (-1.0, 0.0)


def prepare(case, seed):
    s = _State(case)
    shape = (case.get("m"), case.get("n"))
    if case["kind"] == "mlp":
        p, X, y = _make_mlp(case, seed)
        s.model = mxn.nb_mlp_create(s.ctx, p, MLP_LO, MLP_HI)
        s.X, s.y = s.up(X), s.up(y)
        s.grad = torch.zeros(mxn.NB_MLP_PARAMS, dtype=torch.float32, device=s.dev)
        s.loss = torch.zeros(1, dtype=torch.float32, device=s.dev)
        return s
    s.p, s.flags = s.params(), _flags(case)
    if case["kind"] == "batch":
        reps = _make_replicas(case, seed)
        s.f = torch.zeros((3 * sum(r[0] for r in reps), 3), dtype=torch.float32, device=s.dev)
        s.e = torch.zeros((len(reps), 2), dtype=torch.float64, device=s.dev)
        xs, fs, topo, at = [], [], [], 0
        for w, box, first in reps:
            xs.append(s.up(first))
            topo.append(s.topology(w))
            fs.append(s.f[at:at + 3 * w])
            at += 3 * w
            s.grids.append(mxn.nb_grid_sort(s.ctx, box, xs[-1], topo[-1][0], shape))
            s.lists.append(mxn.nb_pairlist_build(s.ctx, s.grids[-1], case["rlist"], -1.0, topo[-1][1], topo[-1][2]))
        s.batch = mxn.nb_batch_create(s.ctx, s.grids, s.lists, xs, fs)
        mxn.nb_batch_set_group(s.batch, 2)
        mxn.nb_batch_bind_topology(s.batch, *[[t[k] for t in topo] for k in range(3)])
        mxn.nb_batch_capture_cycle(s.ctx, s.batch, case["nstlist"], s.p, s.flags, s.e)
        return s
    s.box, first, now = _make_md(case, seed)
    s.first, s.now = s.up(first), [s.up(x) for x in now]
    s.type, s.eo, s.ei = s.topology(case["waters"])
    s.rbb, s.c_bb = _rbb(case, s.box)
    s.f = [torch.zeros((3 * case["waters"], 3), dtype=torch.float32, device=s.dev) for _ in now]
    s.e = torch.zeros((len(now), 2), dtype=torch.float64, device=s.dev)
    s.v = torch.zeros((len(now), 9), dtype=torch.float64, device=s.dev)
    if case["kind"] == "rdf":
        s.bins = 500
        s.hist = torch.zeros((2, 2, s.bins), dtype=torch.int64, device=s.dev)
    if case["kind"] == "recount":
        s.hist = torch.zeros(int(round(RECOUNT_SPAN / RECOUNT_DB)), dtype=torch.float64, device=s.dev)
    s.grids.append(mxn.nb_grid_sort(s.ctx, s.box, s.first, s.type, shape))
    s.lists.append(mxn.nb_pairlist_build(s.ctx, s.grids[0], case["rlist"], s.rbb, s.eo, s.ei))
    return s


def _sort_and_list(s):
    c = s.case
    mxn.nb_grid_sort(s.ctx, s.box, s.first, s.type, (c["m"], c["n"]), s.grids[0])
    mxn.nb_pairlist_build(s.ctx, s.grids[0], c["rlist"], s.rbb, s.eo, s.ei, mxn.NB_LIST_ASYNC, s.lists[0])


def _force_steps(s, lst):
    e, v = s.case["energy"], s.case["virial"]
    for k, x in enumerate(s.now):
        mxn.nb_forces(s.ctx, s.grids[0], lst, x, s.p, s.flags, s.f[k], s.e[k] if e else None, s.v[k] if v else None)
    out = {"f": s.f}
    if e:
        out["e"] = s.e
    if v:
        out["v"] = s.v
    return out


def run(s):
    c = s.case
    if c["kind"] == "mlp":
        mxn.nb_mlp_grad(s.ctx, s.model, s.X, s.y, s.grad, s.loss)
        return {"grad": s.grad, "loss": s.loss}
    if c["kind"] == "batch":
        mxn.nb_batch_replay(s.ctx, s.batch)
        return {"f": s.f, "e": s.e}
    if c["kind"] == "forces":
        return _force_steps(s, s.lists[0])
    if c["kind"] == "cycle":
        _sort_and_list(s)
        return _force_steps(s, s.lists[0])
    if c["kind"] == "prune":
        s.inner = mxn.nb_pairlist_prune(s.ctx, s.lists[0], s.now[0], c["rc"] + 0.05, s.inner)
        return _force_steps(s, s.inner)
    if c["kind"] == "rdf":   # counts add up over the frames of an analysis
        _sort_and_list(s)
        mxn.nb_rdf(s.ctx, s.grids[0], s.lists[0], s.first, c["rc"], s.bins, 2, s.hist)
        return s.hist
    mxn.nb_pairlist_build(s.ctx, s.grids[0], c["rlist"], s.rbb, s.eo, s.ei, 0, s.lists[0])
    mxn.nb_recount(s.ctx, s.grids[0], s.lists[0], s.now[0], s.p, s.c_bb, RECOUNT_DB, s.hist.numel(), s.hist)
    return s.hist


def work(case):
    if case["kind"] == "mlp":
        return {"bytes": 4 * (2 * mxn.NB_MLP_PARAMS + 9 * case["batch"]), "flops": 6 * mxn.NB_MLP_PARAMS * case["batch"]}
    rho = 3.0 * PER_NM3

    def pairs(n, r):
        return n * rho * (4.0 / 3.0) * math.pi * r ** 3 / 2.0

    n = 3 * case["waters"]
    if case["kind"] == "batch":
        n = 3 * sum(r for r in np.rint(np.exp(np.random.default_rng(11).uniform(
            math.log(case["waters"]), math.log(case["largest"]), case["replicas"]))).astype(int).tolist())
    mn = case["m"] * case["n"]
    entries = pairs(n, case["rlist"]) / mn       # cluster pairs, at least
    build = {"bytes": 20 * n + 16 * n + 16 * entries, "flops": 8 * pairs(n, case["rlist"])}
    per_pair = 40 if case["coulomb"] == "rf" else 63
    step = {"bytes": 20 * n + 16 * entries + 12 * n, "flops": per_pair * pairs(n, case["rc"])}
    prune = {"bytes": 16 * n + 32 * entries, "flops": 8 * pairs(n, case["rlist"])}
    read = {"bytes": 20 * n + 16 * entries, "flops": 10 * pairs(n, case["rc"])}
    parts = {"forces": [step], "cycle": [build] + [step] * case["nstlist"], "batch": [build] + [step] * case["nstlist"],
             "prune": [prune] + [step] * case["nstlist"], "rdf": [build, read], "recount": [build, read]}[case["kind"]]
    return {k: float(sum(p[k] for p in parts)) for k in ("bytes", "flops")}


# -------------------------------------------------------- the same in 64 bits

def _pair_terms(case, d, qq, oo, excluded):
    """Force factor F/r, LJ and Coulomb energy of pairs at vectors d (all within rc)."""
    rc, beta = float(np.float32(case["rc"])), float(np.float32(_beta(case["rc"])))
    r2 = (d * d).sum(-1)
    r = r2.sqrt()
    c6, c12 = float(np.float32(C6)), float(np.float32(C12))
    on = oo & ~excluded
    i6 = r2 ** -3
    elj = torch.where(on, (c12 * i6 - c6) * i6 - (c12 / rc ** 6 - c6) / rc ** 6, 0.0)
    flj = torch.where(on, (12.0 * c12 * i6 - 6.0 * c6) * i6 / r2, 0.0)
    one = (~excluded).double()
    if case["coulomb"] == "rf":
        k = 1.0 / (2.0 * rc ** 3)
        return flj + qq * (one / (r2 * r) - 2.0 * k), elj, qq * (one / r + k * r2 - 1.0 / rc - k * rc * rc)
    erfc = torch.special.erfc(beta * r) - 1.0 + one
    g = 2.0 * beta / math.sqrt(math.pi) * torch.exp(-(beta * r) ** 2)
    return flj + qq * (erfc / r + g) / r2, elj, qq * (erfc / r - one * math.erfc(beta * rc) / rc)


def _exact_forces(case, xyzq, box):
    """Forces, (E_LJ, E_Coulomb) and virial of all pairs within rc, by cells no smaller than rc."""
    dev = torch.device("cuda:0" if torch.cuda.is_available() else "cpu")
    L = torch.tensor(box.astype(np.float32).astype(np.float64), device=dev)
    x = torch.from_numpy(xyzq[:, :3].astype(np.float64)).to(dev)
    x = x - torch.floor(x / L) * L
    q = torch.from_numpy(xyzq[:, 3].astype(np.float64)).to(dev)
    n, rc = x.shape[0], float(np.float32(case["rc"]))
    ncell = torch.clamp(torch.floor(L / rc), min=1).long()
    cell3 = torch.minimum((x / L * ncell).long(), ncell - 1)
    cell = (cell3[:, 0] * ncell[1] + cell3[:, 1]) * ncell[2] + cell3[:, 2]
    order = torch.argsort(cell)
    total = int(ncell.prod())
    count = torch.bincount(cell, minlength=total)
    start = torch.cumsum(count, 0) - count
    width = int(count.max())
    slot = torch.arange(n, device=dev) - start[cell[order]]
    table = torch.full((total, width), -1, dtype=torch.long, device=dev)
    table[cell[order], slot] = order
    nx, ny, nz = (int(v) for v in ncell)
    ids = torch.arange(total, device=dev)
    cx, cy, cz = ids // (ny * nz), ids // nz % ny, ids % nz
    around = []   # distinct neighbour cells: all offsets, or every cell of an axis that has fewer than three
    for nn in (nx, ny, nz):
        around.append([-1, 0, 1] if nn >= 3 else list(range(nn)))
    f = torch.zeros((n, 3), dtype=torch.float64, device=dev)
    e = torch.zeros(2, dtype=torch.float64, device=dev)
    v = torch.zeros((3, 3), dtype=torch.float64, device=dev)
    chunk = max(1, int(2e7 // (width * width)))
    coulomb_f = float(np.float32(COULOMB_F))
    for ox in around[0]:
        for oy in around[1]:
            for oz in around[2]:
                other = (((cx + ox) % nx) * ny + (cy + oy) % ny) * nz + (cz + oz) % nz
                for c0 in range(0, total, chunk):
                    ti, tj = table[c0:c0 + chunk], table[other[c0:c0 + chunk]]
                    d = x[ti][:, :, None, :] - x[tj][:, None, :, :]
                    d -= torch.round(d / L) * L
                    near = ((d * d).sum(-1) < rc * rc) & (ti >= 0)[:, :, None] & (tj >= 0)[:, None, :]
                    near &= ti[:, :, None] != tj[:, None, :]
                    b, a, c = torch.nonzero(near, as_tuple=True)
                    i, j, d = ti[b, a], tj[b, c], d[b, a, c]
                    fr, elj, ec = _pair_terms(case, d, coulomb_f * q[i] * q[j], (i % 3 == 0) & (j % 3 == 0),
                                              torch.div(i, 3, rounding_mode="floor") == torch.div(j, 3, rounding_mode="floor"))
                    fd = fr[:, None] * d
                    f.index_add_(0, i, fd)
                    e += 0.5 * torch.stack([elj.sum(), ec.sum()])
                    v += 0.5 * d.T @ fd
    return f.cpu(), e.cpu(), v.reshape(9).cpu()


def _exact_mlp(case, seed):
    p, X, y = (torch.from_numpy(a.astype(np.float64)) for a in _make_mlp(case, seed))
    p.requires_grad_(True)
    w1, b1, w2, b2, w3, b3 = torch.split(p, [512, 64, 4096, 64, 64, 1])
    lo = torch.tensor(np.float32(MLP_LO).astype(np.float64))
    hi = torch.tensor(np.float32(MLP_HI).astype(np.float64))
    h = torch.tanh(((X - lo) * 2.0 / (hi - lo) - 1.0) @ w1.reshape(64, 8).T + b1)
    h = torch.tanh(h @ w2.reshape(64, 64).T + b2)
    loss = ((torch.nn.functional.softplus(h @ w3 + b3, threshold=100.0) - y) ** 2).mean()
    loss.backward()
    return {"grad": p.grad, "loss": loss.detach().reshape(1)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "mlp":
        return _exact_mlp(case, seed)
    if kind in ("rdf", "recount"):   # whole counts; bins of the library's own clusters
        return None
    if kind == "batch":
        got = [_exact_forces(case, first, box) for _, box, first in _make_replicas(case, seed)]
        return {"f": torch.cat([g[0] for g in got]), "e": torch.stack([g[1] for g in got])}
    box, _, now = _make_md(case, seed)
    got = [_exact_forces(case, x, box) for x in now]
    out = {"f": [g[0] for g in got]}
    if case["energy"]:
        out["e"] = torch.stack([g[1] for g in got])
    if case["virial"]:
        out["v"] = torch.stack([g[2] for g in got])
    return out

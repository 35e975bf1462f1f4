"""The work that a user of this library has it do, as cases that can be timed.

A case is one call of the public binding (`paper_2202_01258_amd.qd.Archive`): one or several MAP-Elites
generations on an archive that is already there, the same with the statistics read at the end (a program that
logs its curve), or the creation of an archive (centroids, search structures, first batch).  The sizes are the
repository's own workloads, its batch-size sweep and ablation, and ragged sizes between them.

  listed()         the cases
  draw(rng)        one more case of the same ranges
  prepare(c, s)    the archive a program has in hand, for seed s
  run(state)       one call; returns the batch's and the archive's buffers
  work(c)          bytes and operations one call cannot do without
  tolerance(c)     "exact": every result is defined bit for bit (see tolerance)
  exact(c, s)      the same results worked out in 64 bits with plain torch
"""
from __future__ import annotations

import math

import torch

RASTRIGIN, SPHERE, PROJECTION, POLICY = 0, 1, 2, 3
GRID, CVT = 0, 1
TASKS = {"rastrigin": RASTRIGIN, "sphere": SPHERE, "projection": PROJECTION, "policy": POLICY}
OBS, ACT = 27, 8
BOX = 5.12


# ---------------------------------------------------------------------------
# Cases
# ---------------------------------------------------------------------------
def _testfn(task, n, batch, cells, cvt, init, gens=1, stats=False, samples=0, iters=0):
    """`cells`: bins per side of a grid, or centroids of a CVT.  `init`: "narrow" (genes of the first batch in
    [-0.1, 0.1): the archive starts in a few cells), "wide" (in [-5.12, 5.12)) or "spread" (a level per half)."""
    return {"do": "generations", "task": task, "n": n, "batch": batch, "cells": cells, "cvt": cvt, "init": init,
            "gens": gens, "stats": stats, "samples": samples, "iters": iters}


def _policy(hid, T, batch, cells, gens=1, death=False, stats=False):
    return {"do": "generations", "task": "policy", "hid": hid, "T": T, "batch": batch, "cells": cells, "cvt": True,
            "init": "narrow", "gens": gens, "death": death, "stats": stats, "samples": 0, "iters": 0}


def listed():
    cases = [
        # The smallest calls: one generation of 128 offspring, the paper's low end, where a step is launches and
        # latency.
        dict(_testfn("rastrigin", 100, 128, 100, False, "narrow"), name="rastrigin_grid_b128"),
        # A mid-size batch of short genotypes, all parents in a few cells.
        dict(_testfn("sphere", 100, 16384, 100, False, "narrow"), name="sphere_grid_b16384"),
        # The largest batch of the fixed-budget ablation, started anywhere in the box: every grid cell fills.
        dict(_testfn("rastrigin", 100, 65536, 100, False, "wide"), name="rastrigin_wide_b65536"),
        # The headline configuration: long genotypes, CVT of 10^4 cells, few distinct parents.
        dict(_testfn("projection", 1000, 65536, 10000, True, "narrow"), name="projection_b65536"),
        # The same on a filled archive: parents are distinct rows, thousands of winners early on.
        dict(_testfn("projection", 1000, 65536, 10000, True, "spread"), name="projection_spread_b65536"),
        # Ragged sizes (genotype, batch and cells no multiple of anything), Lloyd centroids, five generations in
        # one call.
        dict(_testfn("projection", 777, 3001, 3003, True, "spread", gens=5, samples=20000, iters=3),
             name="projection_ragged_b3001"),
        # A program that logs its curve: ten generations, then QD-score, coverage and best read on the host.
        dict(_testfn("rastrigin", 100, 1024, 100, False, "wide", gens=10, stats=True), name="rastrigin_logged_b1024"),
        # Policy search at the low end of the batch-size sweep: fewer policies than the card has SIMDs.
        dict(_policy(64, 250, 256, 1024), name="policy64_b256"),
        # Policy search at its ordinary batch.
        dict(_policy(64, 250, 8192, 1024), name="policy64_b8192"),
        # Wider policies that can fail (variable-length episodes), an odd batch.
        dict(_policy(128, 400, 1501, 2500, death=True), name="policy128_death_b1501"),
        # The largest call: wide policies, 1000 steps, 65536 offspring.
        dict(_policy(128, 1000, 65536, 10000), name="policy128_b65536"),
        # A run's start: centroids by Lloyd's algorithm, search structures, first batch evaluated and inserted.
        dict(_testfn("projection", 100, 1024, 10000, True, "spread", samples=100000, iters=5), do="create",
             name="create_cvt_lloyd_c10000"),
    ]
    return cases


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["testfn", "testfn", "testfn", "policy", "policy", "create"])
    if kind == "policy":
        hid = rng.choice([64, 64, 128])
        T = _log_int(rng, 50, 500)
        batch = _log_int(rng, 64, 20000 if hid == 64 else 8000)
        return _policy(hid, T, batch, _log_int(rng, 64, 10000), death=rng.random() < 0.3)
    task = rng.choice(["rastrigin", "sphere", "projection"])
    cvt = task == "projection" or rng.random() < 0.3
    cells = _log_int(rng, 300, 10000)
    if not cvt:
        cells = max(8, int(math.sqrt(cells)))
    init = rng.choice(["narrow", "wide", "spread"])
    if kind == "create":
        return dict(_testfn(task, _log_int(rng, 8, 1000), _log_int(rng, 64, 16384),
                            _log_int(rng, 300, 10000), True, init, samples=_log_int(rng, 5000, 100000),
                            iters=rng.randint(1, 5)), do="create")
    n = _log_int(rng, 100, 1000) if task == "projection" else _log_int(rng, 8, 400)
    return _testfn(task, n, _log_int(rng, 64, 65536), cells, cvt, init, gens=rng.choice([1, 1, 2, 5]),
                   stats=rng.random() < 0.2)


# ---------------------------------------------------------------------------
# What a program holds, and its call
# ---------------------------------------------------------------------------
def _workload(c, seed):
    """The binding's workload dict of a case."""
    w = dict(task=TASKS[c["task"]], tess=CVT if c["cvt"] else GRID, batch=c["batch"], iso_sigma=0.005,
             line_sigma=0.05, init_lo=-0.1, init_hi=0.1, obs=OBS, hid=64, act=ACT, T=1, seed=seed,
             cvt_samples=c["samples"], cvt_iters=c["iters"], death_mode=0, death_below=0.0, init_mode=0)
    if c["task"] == "policy":
        w.update(n=0, D=4, grid=(0, 0, 0, 0), C=c["cells"], lo=(0.0,) * 4, hi=(1.0,) * 4, hid=c["hid"], T=c["T"])
        if c["death"]:
            w.update(death_mode=1, death_below=-0.08)
    else:
        w.update(n=c["n"], D=2, lo=(-BOX, -BOX), hi=(BOX, BOX))
        w.update(grid=(0, 0), C=c["cells"]) if c["cvt"] else w.update(grid=(c["cells"], c["cells"]), C=c["cells"] ** 2)
        if c["init"] == "wide":
            w.update(init_lo=-BOX, init_hi=BOX)
        elif c["init"] == "spread":
            w.update(init_mode=1)
    return w


def _buffers(a):
    """The batch's and the archive's buffers, as a program that reads results holds them."""
    v = a.views()
    out = {k: v[k] for k in ("off_fit", "off_desc", "off_cell", "off_won", "parents", "key", "fit", "desc", "slot",
                             "geno", "occ_list")}
    out["n_occ"] = v["counters"][:1]
    if v["centroids"] is not None:
        out["centroids"] = v["centroids"]
    return out


def prepare(case, seed):
    from paper_2202_01258_amd import qd
    state = {"case": case, "workload": _workload(case, seed), "gen": 1}
    if case["do"] != "create":
        state["archive"] = qd.Archive(state["workload"])
        state["out"] = _buffers(state["archive"])
    return state


def run(state):
    case = state["case"]
    if case["do"] == "create":
        from paper_2202_01258_amd import qd
        a = qd.Archive(state["workload"])
        state["archive"] = a             # the program's archive from here on (the one before is given up)
        return _buffers(a)
    a, k = state["archive"], case["gens"]
    if k == 1:
        a.generation(state["gen"])
    else:
        a.generations(state["gen"], k)
    state["gen"] += k
    if case["stats"]:
        s = a.stats(offset=1000.0)
        return dict(state["out"], qd_score=s["qd_score"], coverage=s["coverage"], best=s["best"])
    return state["out"]


# ---------------------------------------------------------------------------
# What one call cannot do without
# ---------------------------------------------------------------------------
def work(case):
    """Bytes: each parent row that can be distinct read once, each offspring's results and each filled cell's row
    written at most once where most cells change hands (a new archive).  Operations: per gene the generator (10
    rounds of two products and four xors per four genes), the sampler, the variation and the task's term; per
    policy step the multiply-adds."""
    nb, k, D = case["batch"], case["gens"], 4 if case["task"] == "policy" else 2
    cells = case["cells"] if case["cvt"] else case["cells"] ** 2
    if case["task"] == "policy":
        h = case["hid"]
        n = h * OBS + h + h * h + h + ACT * h + ACT
        steps = case["T"] * (0.25 if case["death"] else 1.0)      # failures end episodes early
        per_offspring = 2.0 * steps * (h * OBS + h * h + ACT * h + OBS * OBS + OBS * ACT + ACT) + 30.0 * n
        rows = min(2 * nb, cells)
    else:
        n = case["n"]
        per_offspring = n * (15.0 + 12.0 + 6.0 + (2.0 if case["task"] == "sphere" else 18.0))
        rows = min(2 * nb, cells) if case["init"] != "narrow" else min(2 * nb, 4)
    results = 4 * (1 + D) + 4 + 8 + 1
    if case["do"] == "create":
        points, iters = case["samples"], case["iters"]
        filled = min(nb, cells)
        return {"bytes": float(4 * n * filled + nb * results + 8 * cells * D * (iters + 1)),
                "flops": nb * n * (15.0 + 2.0 + 18.0) + iters * points * (15.0 + 3.0 * D * 9.0)}
    return {"bytes": float(k * (4 * n * rows + nb * results)), "flops": float(k * nb * per_offspring)}


def tolerance(case):
    """Which elite holds a cell is decided by comparing 32-bit objectives, and every later choice follows from it,
    so the library defines each sum's order and each function's arithmetic and its results bit for bit."""
    return "exact"


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain torch
# ---------------------------------------------------------------------------
M32 = 0xffffffff
TAG_INIT, TAG_SELECT, TAG_ISO, TAG_CENTROID, TAG_ENV, TAG_SAMPLE, TAG_LEVEL = range(7)


def _f32(x):
    """A configuration's number as the 32-bit value that the library holds."""
    return float(torch.tensor(x, dtype=torch.float32).item())


def _mul(a, b):
    """Low and high words of a 32 x 32 bit product (a: tensor of words in int64, b: a word)."""
    lo, hi = a & 0xffff, a >> 16
    p, q = lo * b, hi * b                      # below 2^48 each
    return (p + ((q & 0xffff) << 16)) & M32, (q + (p >> 16)) >> 16


def _philox(c0, c1, c2, c3, seed):
    c = list(torch.broadcast_tensors(*[torch.as_tensor(x, dtype=torch.int64, device=_dev()) for x in (c0, c1, c2, c3)]))
    k0, k1 = seed & M32, (seed >> 32) & M32
    for _ in range(10):
        l0, h0 = _mul(c[0], 0xD2511F53)
        l1, h1 = _mul(c[2], 0xCD9E8D57)
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return torch.stack(c, -1)


def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _unit(x):
    return (x >> 8).double() * 2.0 ** -24


def _normal(x):
    p = ((x & 0xffffff) + 1).double() * 2.0 ** -24
    z = -torch.special.ndtri(0.5 * p)
    return torch.where((x >> 31) & 1 == 1, -z, z)


def _genes(item0, items, j, gen, tag, seed):
    """Words of blocks item0 .. item0 + items - 1 of individuals j: [len(j), 4 items]."""
    i = torch.arange(item0, item0 + items, device=_dev())
    return _philox(i[None, :], j[:, None], gen, tag, seed).reshape(len(j), 4 * items)


def _glorot(w):
    o, h, a = OBS, w["hid"], ACT
    lim = [(h * o, math.sqrt(6.0 / (o + h))), (h, 0.0), (h * h, math.sqrt(6.0 / (h + h))), (h, 0.0),
           (a * h, math.sqrt(6.0 / (h + a))), (a, 0.0)]
    return torch.cat([torch.full((k,), v, dtype=torch.float64, device=_dev()) for k, v in lim])


class _Run64:
    """One run of the algorithm in 64 bits."""

    def __init__(self, case, seed):
        self.w, self.seed = _workload(case, seed), seed
        w = self.w
        self.policy = w["task"] == POLICY
        h = w["hid"]
        self.n = h * OBS + h + h * h + h + ACT * h + ACT if self.policy else w["n"]
        self.D, self.C, self.nb = w["D"], w["C"], w["batch"]
        self.lo = torch.tensor([_f32(x) for x in w["lo"]], dtype=torch.float64, device=_dev())
        self.hi = torch.tensor([_f32(x) for x in w["hi"]], dtype=torch.float64, device=_dev())
        self.fit = torch.full((self.C,), math.nan, dtype=torch.float64, device=_dev())
        self.desc = torch.zeros((self.C, self.D), dtype=torch.float64, device=_dev())
        self.geno = torch.zeros((self.C, self.n), dtype=torch.float64, device=_dev())
        self.chunk = max(1, (1 << 26) // max(self.n, 1 if self.policy else 1024))
        if w["tess"] == CVT:
            self.cent = _unit(_philox(torch.arange(self.C, device=_dev()), 0, 0, TAG_CENTROID, seed))[:, :self.D]
            pts = _unit(_philox(torch.arange(w["cvt_samples"], device=_dev()), 0, 0, TAG_SAMPLE, seed))[:, :self.D]
            for _ in range(w["cvt_iters"] if w["cvt_samples"] else 0):
                near = self.nearest(pts)
                count = torch.bincount(near, minlength=self.C).double()
                total = torch.zeros_like(self.cent).index_add_(0, near, pts)
                self.cent = torch.where(count[:, None] > 0, total / count[:, None], self.cent)
        if self.policy:
            e = OBS * (OBS + ACT + 1)
            env = 0.1 * _normal(_philox(torch.arange((e + 3) // 4, device=_dev()), 0, 0, TAG_ENV, seed).reshape(-1)[:e])
            self.A, self.B, self.s0 = torch.split(env, [OBS * OBS, OBS * ACT, OBS])
            self.A, self.B = self.A.view(OBS, OBS).t().contiguous(), self.B.view(OBS, ACT).t().contiguous()
        self.batch(0)

    def nearest(self, u):
        out = []
        for p in u.split(4096):
            d = sum((p[:, None, k] - self.cent[None, :, k]) ** 2 for k in range(self.D))
            out.append(d.argmin(1))
        return torch.cat(out) if out else torch.zeros(0, dtype=torch.int64, device=_dev())

    def first(self, j):
        x = _unit(_genes(0, (self.n + 3) // 4, j, 0, TAG_INIT, self.seed)[:, :self.n])
        w = self.w
        if self.policy:
            a = _glorot(w)
            return x * (2 * a) - a
        lo, hi = _f32(w["init_lo"]), _f32(w["init_hi"])
        x = x * (hi - lo) + lo
        if w["init_mode"]:
            u = _unit(_philox(0, j, 0, TAG_LEVEL, self.seed))
            half = self.n // 2
            x[:, :half] += (u[:, 0] * (self.hi[0] - self.lo[0]) + self.lo[0])[:, None]
            x[:, half:] += (u[:, 1] * (self.hi[1] - self.lo[1]) + self.lo[1])[:, None]
        return x

    def vary(self, j, g):
        x = _philox(0, j, g, TAG_SELECT, self.seed)
        p1, p2 = (self.occ[(x[:, k] * len(self.occ)) >> 32] for k in (0, 1))
        line = _f32(self.w["line_sigma"]) * _normal(x[:, 2])
        e = _normal(_genes(0, (self.n + 3) // 4, j, g, TAG_ISO, self.seed)[:, :self.n])
        a, b = self.geno[p1], self.geno[p2]
        return a + _f32(self.w["iso_sigma"]) * e + line[:, None] * (b - a)

    def evaluate(self, x):
        w = self.w
        if not self.policy:
            term = x * x
            if w["task"] != SPHERE:
                term = term + 20.0 * torch.sin(math.pi * (x - x.round())) ** 2
            fit = -term.sum(1)
            if w["task"] == PROJECTION:
                h = self.n // 2
                d = [x[:, :h].clamp(self.lo[0], self.hi[0]).mean(1), x[:, h:].clamp(self.lo[1], self.hi[1]).mean(1)]
            else:
                d = [x[:, k].clamp(self.lo[k], self.hi[k]) for k in range(2)]
            return fit, torch.stack(d, 1)
        h = w["hid"]
        W1, b1, W2, b2, W3, b3 = torch.split(x, [h * OBS, h, h * h, h, ACT * h, ACT], 1)
        m = len(x)
        W1, W2, W3 = (v.reshape(m, r, k).contiguous() for v, r, k in ((W1, h, OBS), (W2, h, h), (W3, ACT, h)))
        s = self.s0.expand(m, OBS).contiguous()
        fit = torch.zeros(m, dtype=torch.float64, device=_dev())
        desc = torch.zeros((m, 4), dtype=torch.float64, device=_dev())
        valid = torch.zeros(m, dtype=torch.float64, device=_dev())
        alive = torch.ones(m, dtype=torch.bool, device=_dev())
        for _ in range(w["T"]):
            y = torch.tanh(torch.baddbmm(b1[:, :, None], W1, s[:, :, None]))
            y = torch.tanh(torch.baddbmm(b2[:, :, None], W2, y))
            a = torch.tanh(torch.baddbmm(b3[:, :, None], W3, y))[:, :, 0]
            s = torch.tanh(s @ self.A + a @ self.B)
            if w["death_mode"]:
                alive = alive & (s[:, 0] >= _f32(w["death_below"]))
            on = alive.double()
            fit += on * (s[:, 0] - 0.5 * (a * a).sum(1))
            desc += on[:, None] * torch.sigmoid(s[:, 1:5])
            valid += on
        none = valid == 0
        return torch.where(none, math.nan, fit), torch.where(none[:, None], 0.0, desc / valid.clamp(min=1)[:, None])

    def cells(self, desc):
        u = (desc - self.lo) / (self.hi - self.lo)
        if self.w["tess"] == CVT:
            return self.nearest(u)
        bins = torch.tensor(self.w["grid"], device=_dev())
        b = torch.minimum((u * bins).floor().long().clamp(min=0), bins - 1)
        return b[:, 0] * bins[1] + b[:, 1]

    def make(self, j, g):
        return self.first(j) if g == 0 else self.vary(j, g)

    def batch(self, g):
        parts = torch.arange(self.nb, device=_dev()).split(self.chunk)
        got = [self.evaluate(self.make(j, g)) for j in parts]
        fit, desc = (torch.cat([x[k] for x in got]) for k in (0, 1))
        ok = ~fit.isnan()
        cell = self.cells(desc)
        # the best offspring of each cell, the first of equal ones
        order = torch.argsort(torch.where(ok, fit, -math.inf), descending=True, stable=True)
        order = order[ok[order]]
        first = torch.full((self.C,), self.nb, dtype=torch.int64, device=_dev())
        first.scatter_reduce_(0, cell[order], torch.arange(len(order), device=_dev()), "amin")
        won = (first < self.nb).nonzero()[:, 0]
        j = order[first[won]]
        keep = self.fit[won].isnan() | (fit[j] > self.fit[won])
        won, j = won[keep], j[keep]
        if len(j):
            new = torch.cat([self.make(p, g) for p in j.split(self.chunk)])
            self.geno[won], self.fit[won], self.desc[won] = new, fit[j], desc[j]
        self.occ = (~self.fit.isnan()).nonzero()[:, 0]
        self.off_fit, self.off_desc = fit, desc


def exact(case, seed):
    w = _workload(case, seed)
    if case["task"] == "policy" and w["T"] * w["batch"] * w["hid"] ** 2 > 2e11:
        return None                                               # more than 20 s
    r = _Run64(case, seed)
    for g in range(1, 1 + (0 if case["do"] == "create" else case["gens"])):
        r.batch(g)
    out = {k: None for k in ("off_cell", "off_won", "parents", "key", "slot", "geno", "occ_list", "n_occ")}
    out.update(off_fit=r.off_fit, off_desc=r.off_desc, fit=r.fit, desc=r.desc)
    if case["cvt"]:
        out["centroids"] = r.cent
    if case["stats"]:
        filled = r.fit[r.occ]
        out.update(qd_score=float((filled + 1000.0).sum()), coverage=len(r.occ) / r.C, best=float(filled.max()))
    return out

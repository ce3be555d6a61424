"""Performance cases of the MCPT(2) solves, through the package's public calls.

A case is a cluster of monomers on a simple cubic lattice (nx x ny x nz sites, 3.4 Angstrom, open
boundaries, pairs within the squared cutoff in spacings) with random orbital energies and integrals
of the magnitudes of the HF-crystal workloads (see the draws below), and one of the calls a program
makes on it:

  solve      mcpt_run of a resident problem, then its energies and amplitudes
  batch      the same for clusters of uneven size uploaded as one batch
  singles    mcpt_singles of a resident problem
  lccd       mcpt_run with the intramonomer integrals attached (full monomer equation)
  dimer      mcpt_run with the intramonomer and the dimer classes attached
  displaced  a displaced geometry made on the device from a resident crystal, solved from the
             crystal's amplitudes and released (one point of a finite-difference grid)
  served     requests on host data submitted together, waited for, read and released

`exact` gives the same results as plain torch products in 64 bits.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_1409_2700_amd as mc

SCALE = 0.18              # coupling scale of the V blocks: about 15 sweeps to 1e-10
PRECISION = {"fp64": mc.MCPT_FP64, "fp32": mc.MCPT_FP32, "bf16": mc.MCPT_BF16}
# monomer sizes (occupied, virtual): the HF molecule's basis and a larger one, and the odd sizes the tests use
POOLS = {
    "two": [(5, 27), (8, 56)],
    "ragged": [(1, 1), (2, 3), (3, 17), (4, 9), (5, 27), (6, 21), (4, 31)],
}
FIELDS = dict(kind="solve", nx=2, ny=2, nz=2, cutoff2=9, pool="one", o=5, v=27, precision="fp64", tol=1e-10,
              deterministic=0, graph=0, clusters=1, smallest=0, largest=0)


def listed():
    case = lambda name, **kw: dict(FIELDS, name=name, **kw)
    return [
        # the smallest crystal: every pair on a compute unit of its own, launches and host checks count
        case("cube8", nx=2, ny=2, nz=2, cutoff2=12),
        # a mid-size crystal: a handful of pairs per compute unit
        case("cube125", nx=5, ny=5, nz=5, cutoff2=4),
        # the 1000-monomer crystal of the benchmark, 42,144 pairs
        case("cube1000", nx=10, ny=10, nz=10, cutoff2=9),
        # the same crystal with BF16 pair products and the FP64 polish, at the tolerance of the displacement grids
        case("cube1000-bf16", nx=10, ny=10, nz=10, cutoff2=9, precision="bf16", tol=1e-12),
        # a batch of uneven clusters of o5v27 and o8v56 monomers (blocks too large for LDS), FP64 with a graph
        case("batch-fp64", kind="batch", cutoff2=4, pool="two", clusters=3, smallest=20, largest=64, graph=1),
        # the same batch with FP32 pair products and the polish
        case("batch-fp32", kind="batch", cutoff2=4, pool="two", clusters=3, smallest=20, largest=64, graph=1,
             precision="fp32", tol=1e-12),
        # monomers of odd sizes down to one orbital pair, bitwise-repeatable accumulation
        case("ragged-det", nx=4, ny=4, nz=5, cutoff2=4, pool="ragged", deterministic=1),
        # singles on the 1000-monomer crystal
        case("singles1000", kind="singles", nx=10, ny=10, nz=10, cutoff2=9),
        # full monomer equation
        case("lccd216", kind="lccd", nx=6, ny=6, nz=6, cutoff2=2),
        # dimer-internal terms on a nearest-neighbour crystal
        case("dimer216", kind="dimer", nx=6, ny=6, nz=6, cutoff2=1),
        # one displaced geometry of a finite-difference grid
        case("displaced343", kind="displaced", nx=7, ny=7, nz=7, cutoff2=4, tol=1e-12),
        # requests of uneven size arriving together, from host memory
        case("served", kind="served", cutoff2=9, clusters=6, smallest=8, largest=64),
    ]


def draw(rng):
    """A case of the listed ranges: 8 to 1000 monomers, cutoffs of 1 to 3 spacings, o 2..8, v 5..56."""
    while True:
        c = dict(FIELDS, kind=rng.choice(["solve", "solve", "solve", "solve", "batch", "singles", "lccd", "dimer",
                                          "displaced", "served"]))
        n = round(math.exp(rng.uniform(math.log(8), math.log(1000))))
        c["nx"] = max(1, round(n ** (1 / 3) * rng.uniform(0.7, 1.3)))
        c["ny"] = max(1, round(math.sqrt(n / c["nx"]) * rng.uniform(0.8, 1.25)))
        c["nz"] = max(2, round(n / (c["nx"] * c["ny"])))
        c["cutoff2"] = rng.choice([1, 2, 3, 4, 5, 8, 9])
        if rng.random() < 0.5:
            c["o"], c["v"] = rng.randint(2, 8), round(math.exp(rng.uniform(math.log(5), math.log(56))))
        if c["kind"] in ("solve", "batch"):
            c["precision"] = rng.choice(["fp64", "fp64", "fp64", "bf16", "fp32"])
            c["tol"] = 1e-10 if c["precision"] == "fp64" else 1e-12
            c["graph"] = rng.choice([0, 1])
            c["pool"] = rng.choice(["one", "one", "two", "ragged"])
            if c["kind"] == "solve" and not c["graph"]:
                c["deterministic"] = rng.choice([0, 0, 1])
        if c["kind"] == "displaced":
            c["tol"] = 1e-12
        if c["kind"] in ("lccd", "dimer"):
            c["o"], c["v"] = rng.choice([(5, 27), (rng.randint(2, 6), rng.randint(6, 32))])
        if c["kind"] in ("batch", "served"):
            c["clusters"] = rng.randint(2, 6)
            c["smallest"] = rng.randint(4, 24)
            c["largest"] = rng.randint(25, 96)
            c["nx"] = c["ny"] = c["nz"] = 0
        if c["pool"] == "two":
            c["cutoff2"] = min(c["cutoff2"], 4)
        w = work(c)
        top = {"lccd": 4e12, "dimer": 4e12, "served": 4e12, "displaced": 4e12}.get(c["kind"], 12e12)
        floor = 1e6
        if c["kind"] == "dimer":
            shape = _shape(c)
            if len(shape.pairs) * c["v"] ** 4 * 8 > 6e9:
                continue
        if c["precision"] == "fp32":
            top = 6e12
        if c["deterministic"]:
            top = 6e12
        if floor < w["flops"] <= top and len(_shape(c).pairs) > 0:
            return c


# ---- shapes ---------------------------------------------------------------------------------------
def _sites(nx, ny, nz):
    g = np.stack(np.meshgrid(np.arange(nx), np.arange(ny), np.arange(nz), indexing="ij"), -1)
    return g.reshape(-1, 3).astype(np.int64)


def _pairs(sites, cutoff2):
    i, j = np.triu_indices(len(sites), 1)
    d2 = ((sites[i] - sites[j]) ** 2).sum(1)
    keep = d2 <= cutoff2
    return np.stack([i[keep], j[keep]], 1).astype(np.int32), d2[keep].astype(np.float64)


def _cluster_sizes(c):
    """Monomer counts of the clusters of a batch or of the requests, log-spaced."""
    n = c["clusters"]
    step = math.log(c["largest"] / c["smallest"]) / max(1, n - 1)
    return [round(c["smallest"] * math.exp(step * k)) for k in range(n)]


def _one_shape(c, sites, first):
    n = len(sites)
    if c["pool"] == "one":
        sizes = [(c["o"], c["v"])] * n
    else:
        pool = POOLS[c["pool"]]
        sizes = [pool[((first + x) * 7919 + 13) % 101 % len(pool)] for x in range(n)]
    pairs, d2 = _pairs(sites, c["cutoff2"])
    return SimpleNamespace(sizes=np.array(sizes, dtype=np.int64).reshape(-1, 2), pairs=pairs, d2=d2)


def _shapes(c):
    """The clusters of a case (one, or those of a batch or of the requests)."""
    if c["kind"] not in ("batch", "served"):
        return [_one_shape(c, _sites(c["nx"], c["ny"], c["nz"]), 0)]
    out, first = [], 0
    for n in _cluster_sizes(c):
        side = 1
        while side ** 3 < n:
            side += 1
        out.append(_one_shape(c, _sites(side, side, side)[:n], first))
        first += n
    return out


def _shape(c):
    """All clusters of a case as one, the pair indices shifted."""
    parts = _shapes(c)
    at = np.concatenate([[0], np.cumsum([len(p.sizes) for p in parts])])
    return SimpleNamespace(sizes=np.concatenate([p.sizes for p in parts]),
                           pairs=np.concatenate([p.pairs + np.int32(a) for p, a in zip(parts, at)]),
                           d2=np.concatenate([p.d2 for p in parts]))


def work(c):
    """Bytes of the inputs and results, each once, and the operations of the usual number of sweeps (14 of the
    doubles, 6 from a neighbouring geometry's amplitudes, 30 of the singles, 22 + 25 of the full monomer equation)."""
    s = _shape(c)
    n = s.sizes[:, 0] * s.sizes[:, 1]
    nx, ny = n[s.pairs[:, 0]].astype(float), n[s.pairs[:, 1]].astype(float)
    v = float((nx * ny).sum())
    t = float((n.astype(float) ** 2).sum())
    values = v + 2 * t + float(s.sizes.sum()) + len(s.pairs) + 2 * len(n)
    sweep = float((4 * nx * ny * (nx + ny)).sum()) + 12 * t
    if c["kind"] == "singles":
        return {"bytes": 8.0 * (v + 3 * float(n.sum())), "flops": 30 * 4 * v}
    if c["kind"] in ("lccd", "dimer"):
        o, vv = float(c["o"]), float(c["v"])
        ladder = len(n) * (2 * o ** 2 * vv ** 4 + 2 * o ** 4 * vv ** 2)
        rings = len(n) * 6 * (o * vv) ** 3
        values += len(n) * (vv ** 4 + o ** 4 + o ** 2 * vv ** 2)
        flops = 14 * sweep + 40 * (ladder + rings)
        if c["kind"] == "dimer":
            values += len(nx) * (vv ** 4 + o ** 4 + 2 * o ** 2 * vv ** 2)
            flops += 25 * len(nx) * (2 * o ** 2 * vv ** 4 + 8 * (o * vv) ** 3)
        return {"bytes": 8.0 * values, "flops": flops}
    return {"bytes": 8.0 * values, "flops": (6 if c["kind"] == "displaced" else 14) * sweep}


# ---- draws ----------------------------------------------------------------------------------------
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _draw(shape, gen, dev, k_scale=1.0):
    """Inputs of one cluster: occupied energies U[-1.5, -0.5], virtual U[0.2, 3.0], K = <ab|ij> N(0, 0.05^2)
    antisymmetrised in (i,j) and (a,b), V = (ai|bj) N(0, (0.18 * 0.05 / R^3)^2) with R in spacings."""
    kw = dict(generator=gen, device=dev, dtype=torch.float64)
    sizes = [(int(o), int(v)) for o, v in shape.sizes]
    one = len(set(sizes)) == 1
    n = np.array([o * v for o, v in sizes])
    blocks = [(len(sizes), *sizes[0])] if one else [(1, o, v) for o, v in sizes]
    eps, ks = [], []
    for count, o, v in blocks:
        eo = torch.sort(torch.rand(count, o, **kw), 1)[0] - 1.5
        ev = torch.sort(torch.rand(count, v, **kw), 1)[0] * 2.8 + 0.2
        eps.append(torch.cat([eo, ev], 1).reshape(-1))
        g = torch.randn(count, o, o, v, v, **kw) * (0.05 * k_scale)
        g = g - g.transpose(1, 2)
        ks.append((0.5 * (g - g.transpose(3, 4))).reshape(-1))
    per = n[shape.pairs[:, 0]].astype(np.int64) * n[shape.pairs[:, 1]]
    # the couplings of blocks larger than the HF molecule's are scaled down, so that the sweeps still converge
    big = SCALE * np.minimum(1.0, np.sqrt(135.0 / np.maximum(1, n.max()))) if one else SCALE
    sigma = torch.from_numpy(big * 0.05 / shape.d2 ** 1.5).to(dev)
    v = torch.randn(int(per.sum()), **kw)
    if one:
        v.view(len(per), -1).mul_(sigma[:, None])
    else:
        v.mul_(torch.repeat_interleave(sigma, torch.from_numpy(per).to(dev)))
    return SimpleNamespace(n_occ=np.array([o for o, _ in sizes], dtype=np.int32),
                           n_vir=np.array([w for _, w in sizes], dtype=np.int32), sizes=sizes, n=n, pairs=shape.pairs,
                           d2=shape.d2, eps=torch.cat(eps), k=torch.cat(ks), v=v)


def _average(g, first, perms, sigma):
    """Draws averaged over permutations of the axes after the first, an element's deviation kept at sigma."""
    s = g.clone()
    for p in perms[1:]:
        s += g.permute(0, *[1 + q for q in p])
    return s * (sigma / math.sqrt(len(perms)))


_EIGHT = [(0, 1, 2, 3), (1, 0, 2, 3), (0, 1, 3, 2), (1, 0, 3, 2), (2, 3, 0, 1), (3, 2, 0, 1), (2, 3, 1, 0), (3, 2, 1, 0)]
_FOUR = _EIGHT[:4]


def _intramonomer(c, count, gen, dev):
    """<ab|cd>, <ij|kl> and (ij|ab) of every monomer at sigma 0.01, with the symmetry of real orbitals."""
    o, v = c["o"], c["v"]
    kw = dict(generator=gen, device=dev, dtype=torch.float64)
    w = _average(torch.randn(count, v, v, v, v, **kw), 1, _EIGHT, 0.01).permute(0, 1, 3, 2, 4).contiguous()
    q = _average(torch.randn(count, o, o, o, o, **kw), 1, _EIGHT, 0.01).permute(0, 1, 3, 2, 4).contiguous()
    j = _average(torch.randn(count, o, o, v, v, **kw), 1, _FOUR, 0.01).contiguous()
    return w, q, j


def _dimer_classes(c, d2, gen, dev):
    """The four dimer classes of every pair at sigma 0.01 / R^3, symmetric within each charge distribution."""
    o, v, P = c["o"], c["v"], len(d2)
    kw = dict(generator=gen, device=dev, dtype=torch.float64)
    s = torch.from_numpy(d2 ** -1.5).to(dev)[:, None, None, None, None]
    w = (_average(torch.randn(P, v, v, v, v, **kw), 1, _FOUR, 0.01) * s).permute(0, 1, 3, 2, 4).contiguous()
    q = (_average(torch.randn(P, o, o, o, o, **kw), 1, _FOUR, 0.01) * s).permute(0, 1, 3, 2, 4).contiguous()
    cx = (_average(torch.randn(P, o, o, v, v, **kw), 1, _FOUR, 0.01) * s).contiguous()
    cy = (_average(torch.randn(P, o, o, v, v, **kw), 1, _FOUR, 0.01) * s).contiguous()
    return w, q, cx, cy


def _inputs(c, seed):
    """Every input of a case, made from the seed alone."""
    dev = _device()
    gen = torch.Generator(device=dev).manual_seed(seed)
    k_scale = 0.2 if c["kind"] in ("lccd", "dimer") else 1.0
    probs = [_draw(s, gen, dev, k_scale) for s in _shapes(c)]
    more = SimpleNamespace(w=None, intra=None, dimer=None, moved=None)
    p = probs[0]
    if c["kind"] == "singles":
        more.w = torch.randn(int(p.n.sum()), generator=gen, device=dev, dtype=torch.float64) * 0.05
    if c["kind"] in ("lccd", "dimer"):
        more.intra = _intramonomer(c, len(p.sizes), gen, dev)
    if c["kind"] == "dimer":
        more.dimer = _dimer_classes(c, p.d2, gen, dev)
    if c["kind"] == "displaced":   # one monomer moved by 0.01 Angstrom along x: its pairs' blocks times (R0 / R)^3
        sites = _sites(c["nx"], c["ny"], c["nz"]).astype(np.float64)
        at = seed % len(sites)
        mine = np.nonzero((p.pairs == at).any(1))[0]
        other = np.where(p.pairs[mine, 0] == at, p.pairs[mine, 1], p.pairs[mine, 0])
        d = sites[at] - sites[other]
        r0 = np.sqrt((d ** 2).sum(1))
        d[:, 0] += 0.01 / 3.4
        more.moved = (mine.astype(np.int64), (r0 / np.sqrt((d ** 2).sum(1))) ** 3)
    return probs, more


# ---- the calls ------------------------------------------------------------------------------------
_context = None


def _ctx():
    global _context
    if _context is None:
        _context = mc.Context(0)
    return _context


class _Resident:
    """A resident problem, released with the object that a program keeps for it."""

    def __init__(self, ctx, pid):
        self.ctx, self.pid = ctx, pid

    def __del__(self):
        try:
            self.ctx.release(self.pid)
        except Exception:
            pass


def _host(p):
    """The arrays of a cluster on the host, as a program that read or computed its integrals there has them."""
    return mc.HostProblem(SimpleNamespace(n_occ=p.n_occ, n_vir=p.n_vir, eps=p.eps.cpu().numpy(), k=p.k.cpu().numpy(),
                                          pairs=p.pairs, v=p.v.cpu().numpy()))


def _options(c):
    return dict(tol=c["tol"], precision=PRECISION[c["precision"]], deterministic=c["deterministic"], graph=c["graph"])


def prepare(c, seed):
    probs, more = _inputs(c, seed)
    torch.cuda.synchronize()
    ctx = _ctx()
    st = SimpleNamespace(case=c, ctx=ctx, opts=_options(c), problem=None, w=None, host=None, moved=more.moved, t=None)
    if c["kind"] == "served":
        st.host = [_host(p) for p in probs]
        return st
    if c["kind"] == "batch":
        st.problem = _Resident(ctx, ctx.upload_batch([_host(p) for p in probs]))
        return st
    p = probs[0]
    st.problem = _Resident(ctx, ctx.upload_device(p.n_occ, p.n_vir, p.pairs, p.eps.data_ptr(), p.k.data_ptr(),
                                                  p.v.data_ptr()))
    if more.intra is not None:
        ctx.lccd_attach(st.problem.pid, None, device_ptrs=tuple(t.data_ptr() for t in more.intra))
    if more.dimer is not None:
        ctx.dimer_attach(st.problem.pid, None, device_ptrs=tuple(t.data_ptr() for t in more.dimer))
    if more.w is not None:
        st.w = more.w.cpu().numpy()
    if c["kind"] == "displaced":   # the crystal's own solve, whose amplitudes the points start from
        ctx.run(st.problem.pid, **st.opts)
        st.t = ctx.energy(st.problem.pid)["t"]
    return st


def _results(ctx, pid, s, fp64):
    """What a solve gives.  The sweeps of a reduced-precision solve are no result (they depend on its rounding)."""
    out = ctx.energy(pid)
    out["total"] = np.array([s["e_total"], s["e_mono"], s["e_dimer"], s["e_mono0"]])
    if fp64:
        out["sweeps"] = s["sweeps"]
    return out


def run(st):
    ctx, kind = st.ctx, st.case["kind"]
    fp64 = st.case["precision"] == "fp64"
    if kind == "served":
        tickets = [ctx.submit(h, **st.opts) for h in st.host]
        out = []
        for t in tickets:
            s = ctx.wait(t)
            if s["status"] != mc.MCPT_OK:
                raise RuntimeError(s["error"])
            out.append(_results(ctx, t, s, True))
            ctx.release(t)
        return out
    if kind == "singles":
        s = ctx.singles(st.problem.pid, st.w, tol=st.case["tol"])
        out = ctx.singles_result(st.problem.pid)
        out["total"] = np.array([s["e_m1"], s["e_m1_0"]])
        out["sweeps"] = s["sweeps"]
        return out
    if kind == "displaced":
        pid = ctx.upload_scaled(st.problem.pid, *st.moved)
        out = _results(ctx, pid, ctx.run(pid, warm_t=st.t, **st.opts), False)
        ctx.release(pid)
        return out
    s = ctx.run(st.problem.pid, **st.opts)
    out = _results(ctx, st.problem.pid, s, fp64)
    if kind == "batch":   # clusters stop by themselves: their own summaries
        out["clusters"] = np.array([[q["e_total"], q["e_mono"], q["e_dimer"], q["e_mono0"]]
                                    for q in ctx.cluster_results(st.problem.pid)])
    if kind == "dimer":
        out["tau"] = ctx.dimer_tau(st.problem.pid)
    return out


# ---- the same in plain torch, 64 bits -------------------------------------------------------------
class _Plain:
    """Doubles amplitudes of one cluster by Jacobi sweeps; matrices T[(i,a),(j,b)], monomers grouped by size."""

    def __init__(self, p):
        self.p, dev = p, p.v.device
        kinds = sorted(set(p.sizes))
        self.kinds = kinds
        of = [kinds.index(s) for s in p.sizes]
        self.place, self.members = [], [[] for _ in kinds]
        for x, g in enumerate(of):
            self.place.append((g, len(self.members[g])))
            self.members[g].append(x)
        eoff = np.concatenate([[0], np.cumsum([o + v for o, v in p.sizes])])
        koff = np.concatenate([[0], np.cumsum([(o * v) ** 2 for o, v in p.sizes])])
        self.K, self.d = [], []
        for g, (o, v) in enumerate(kinds):
            if len(kinds) == 1:
                k = p.k.view(-1, o, o, v, v)
                e = p.eps.view(-1, o + v)
            else:
                k = torch.stack([p.k[koff[x]:koff[x + 1]].view(o, o, v, v) for x in self.members[g]])
                e = torch.stack([p.eps[eoff[x]:eoff[x + 1]] for x in self.members[g]])
            self.K.append(k.permute(0, 1, 3, 2, 4).reshape(-1, o * v, o * v).contiguous())
            self.d.append((e[:, :o, None] - e[:, None, o:]).reshape(-1, o * v))
        voff = np.concatenate([[0], np.cumsum(p.n[p.pairs[:, 0]].astype(np.int64) * p.n[p.pairs[:, 1]])])
        by = {}
        for q, (x, y) in enumerate(p.pairs):
            by.setdefault((of[x], of[y]), []).append(q)
        self.parts = []
        for (gx, gy), qs in by.items():
            nx, ny = (kinds[g][0] * kinds[g][1] for g in (gx, gy))
            for a in range(0, len(qs), 2048):
                some = qs[a:a + 2048]
                if len(by) == 1:
                    V = p.v[voff[some[0]]:voff[some[-1] + 1]].view(-1, nx, ny)
                else:
                    V = torch.stack([p.v[voff[q]:voff[q + 1]].view(nx, ny) for q in some])
                ix = torch.tensor([self.place[p.pairs[q, 0]][1] for q in some], device=dev)
                iy = torch.tensor([self.place[p.pairs[q, 1]][1] for q in some], device=dev)
                self.parts.append((gx, gy, torch.tensor(some, device=dev), ix, iy, V))
        self.D = [1.0 / (d[:, :, None] + d[:, None, :]) for d in self.d]

    def swap(self, g, T):
        o, v = self.kinds[g]
        return T.view(-1, o, v, o, v).transpose(1, 3).reshape(T.shape)

    def adapted(self, T):
        return [2.0 * t - self.swap(g, t) for g, t in enumerate(T)]

    def tau(self, part, M, internal=None):
        gx, gy, _, ix, iy, V = part
        s = V + torch.bmm(M[gx][ix], V) + torch.bmm(V, M[gy][iy].transpose(1, 2).contiguous())
        if internal is not None:
            s = s + internal
        return s / (self.d[gx][ix][:, :, None] + self.d[gy][iy][:, None, :])

    def pair_sum(self, taus):
        G = [torch.zeros_like(k) for k in self.K]
        for (gx, gy, _, ix, iy, V), tau in taus:
            G[gx].index_add_(0, ix, torch.bmm(tau, V.transpose(1, 2).contiguous()))
            G[gy].index_add_(0, iy, torch.bmm(tau.transpose(1, 2).contiguous(), V))
        return [2.0 * (g + g.transpose(1, 2)) for g in G]

    def first(self):
        return [d * k for d, k in zip(self.D, self.K)]

    def e_m2(self, T):
        e = torch.empty(len(self.p.sizes), dtype=torch.float64, device=self.p.v.device)
        for g, (k, m) in enumerate(zip(self.K, self.adapted(T))):
            e[torch.tensor(self.members[g], device=e.device)] = (k * m).sum((1, 2))
        return e

    def e_d2(self, taus):
        e = torch.zeros(len(self.p.pairs), dtype=torch.float64, device=self.p.v.device)
        for part, tau in taus:
            e[part[2]] = 4.0 * (part[5] * tau).sum((1, 2))
        return e

    def flat(self, T):
        """T[i][j][a][b], monomers in their order."""
        if len(self.kinds) == 1:
            o, v = self.kinds[0]
            return T[0].view(-1, o, v, o, v).permute(0, 1, 3, 2, 4).reshape(-1)
        out = []
        for g, i in self.place:
            o, v = self.kinds[g]
            out.append(T[g][i].view(o, v, o, v).permute(0, 2, 1, 3).reshape(-1))
        return torch.cat(out)


def _iterate(step, T, tol, most=500):
    for k in range(most):
        new = step(T)
        r = max(float((a - b).abs().max()) for a, b in zip(new, T))
        T = new
        if r < tol:
            return T, k + 1
    raise RuntimeError("not converged")


def _exact_doubles(p, tol):
    s = _Plain(p)

    def step(T):
        M = s.adapted(T)
        return [d * (k + g) for d, k, g in zip(s.D, s.K, s.pair_sum((part, s.tau(part, M)) for part in s.parts))]

    first = s.first()
    T, sweeps = _iterate(step, first, tol)
    M = s.adapted(T)
    e_d2 = s.e_d2((part, s.tau(part, M)) for part in s.parts)
    return _laid_out(s, T, s.e_m2(T), s.e_m2(first), e_d2, sweeps)


def _laid_out(s, T, e_m2, e_0, e_d2, sweeps):
    e_mono, e_dimer = float(e_m2.sum()), float(e_d2.sum())
    return dict(e_m2=e_m2.cpu().numpy(), de_m2=(e_m2 - e_0).cpu().numpy(), e_d2=e_d2.cpu().numpy(),
                t=s.flat(T).cpu().numpy(), total=np.array([e_mono + e_dimer, e_mono, e_dimer, float(e_0.sum())]),
                sweeps=sweeps)


def _exact_full(c, p, more):
    """Full monomer equation, with the dimer-internal terms where their classes are given (one monomer size)."""
    s = _Plain(p)
    o, v, N = c["o"], c["v"], len(p.sizes)
    W, Q, J = more.intra
    n = o * v
    K = p.k.view(N, o, o, v, v)
    W2 = W.reshape(N, v * v, v * v).transpose(1, 2).contiguous()
    Q2 = Q.reshape(N, o * o, o * o).transpose(1, 2).contiguous()
    hat = lambda A: A.permute(0, 1, 3, 2, 4).reshape(N, n, n).contiguous()        # [i,j,a,b] -> [(i,a),(j,b)]
    ring_k, ring_j = hat(K), hat(J.transpose(1, 2).contiguous())
    vswap = lambda A: A.view(N, o, v, o, v).transpose(2, 4).reshape(N, n, n)

    def intra(T):
        t4 = T.view(N, o, v, o, v).permute(0, 1, 3, 2, 4).contiguous()
        lad = torch.bmm(t4.view(N, o * o, v * v), W2) + torch.bmm(Q2, t4.view(N, o * o, v * v))
        M = 2.0 * T - s.swap(0, T)
        R = torch.bmm(ring_k, M) - torch.bmm(ring_j, T) - vswap(torch.bmm(ring_j, vswap(T).contiguous()))
        return hat(lad.view(N, o, o, v, v)) + R + R.transpose(1, 2)

    T0 = s.first()
    iso, _ = _iterate(lambda T: [s.D[0] * (s.K[0] + intra(T[0]))], T0, c["tol"])
    e_0 = s.e_m2(iso)
    P = len(p.pairs)
    state = SimpleNamespace(tau=None)

    def dimer_terms(part, tau):
        _, _, q, ix, iy, _ = part
        Wd, Qd, CX, CY = (a[q] for a in more.dimer)
        b = len(q)
        t = tau.view(b, o, v, o, v)
        t4 = t.permute(0, 1, 3, 2, 4).reshape(b, o * o, v * v).contiguous()                  # [(i,j),(a,b)]
        lad = torch.bmm(t4, Wd.reshape(b, v * v, v * v).transpose(1, 2).contiguous())
        lad = lad + torch.bmm(Qd.reshape(b, o * o, o * o).transpose(1, 2).contiguous(), t4)
        out = lad.view(b, o, o, v, v).permute(0, 1, 3, 2, 4).reshape(b, n, n)
        # -C_X[k,i,b,c] tau[k,a,j,c] and -C_Y[k,j,a,c] tau[i,c,k,b]
        cx = CX.permute(0, 2, 3, 1, 4).reshape(b, n, n).contiguous()                          # [(i,b),(k,c)]
        t1 = t.permute(0, 1, 4, 3, 2).reshape(b, n, n).contiguous()                           # [(k,c),(j,a)]
        out = out - torch.bmm(cx, t1).view(b, o, v, o, v).permute(0, 1, 4, 3, 2).reshape(b, n, n)
        cy = CY.permute(0, 2, 3, 1, 4).reshape(b, n, n).contiguous()                          # [(j,a),(k,c)]
        t2 = t.permute(0, 3, 2, 1, 4).reshape(b, n, n).contiguous()                           # [(k,c),(i,b)]
        out = out - torch.bmm(cy, t2).view(b, o, v, o, v).permute(0, 3, 2, 1, 4).reshape(b, n, n)
        A = 2.0 * ring_k - ring_j
        return out + torch.bmm(A[ix], tau) + torch.bmm(tau, A[iy].transpose(1, 2).contiguous())

    def taus(T):
        M = s.adapted(T)
        old = state.tau
        if more.dimer is None:
            return ((part, s.tau(part, M)) for part in s.parts)
        return [(part, s.tau(part, M, None if old is None else dimer_terms(part, old[k]))) for k, part in
                enumerate(s.parts)]

    def step(T):
        got = taus(T)
        if more.dimer is not None:
            state.tau = [t for _, t in got]
        return [s.D[0] * (s.K[0] + s.pair_sum(got)[0] + intra(T[0]))]

    T, sweeps = _iterate(step, T0, c["tol"])
    got = list(taus(T))
    out = _laid_out(s, T, s.e_m2(T), e_0, s.e_d2(got), sweeps)
    if more.dimer is not None:
        tau = torch.empty(P, n, n, dtype=torch.float64, device=p.v.device)
        for part, t in got:
            tau[part[2]] = t
        out["tau"] = tau.reshape(-1).cpu().numpy()
    return out


def _exact_singles(c, p, w):
    o, v = p.sizes[0]
    n, N = o * v, len(p.sizes)
    e = p.eps.view(N, o + v)
    d = (e[:, :o, None] - e[:, None, o:]).reshape(N, n)
    x, y = (torch.from_numpy(p.pairs[:, k].astype(np.int64)).to(w.device) for k in (0, 1))
    V = p.v.view(-1, n, n)
    w = w.view(N, n)

    def step(T):
        u = torch.zeros_like(w)
        for a in range(0, len(V), 8192):
            b = slice(a, a + 8192)
            u.index_add_(0, x[b], torch.bmm(V[b], T[0][y[b]][:, :, None])[:, :, 0])
            u.index_add_(0, y[b], torch.bmm(T[0][x[b]][:, None, :], V[b])[:, 0, :])
        return [(w + 2.0 * u) / d]

    first = w / d
    T, sweeps = _iterate(step, [first], c["tol"])
    e1, e0 = 2.0 * (w * T[0]).sum(1), 2.0 * (w * first).sum(1)
    return dict(e_m1=e1.cpu().numpy(), t1=T[0].reshape(-1).cpu().numpy(),
                total=np.array([float(e1.sum()), float(e0.sum())]), sweeps=sweeps)


def exact(c, seed):
    if not torch.cuda.is_available():
        return None
    probs, more = _inputs(c, seed)
    fp64 = c["precision"] == "fp64" and c["kind"] != "displaced"
    tol = c["tol"] if fp64 else 1e-15
    if c["kind"] == "singles":
        return _exact_singles(c, probs[0], more.w)
    if c["kind"] in ("lccd", "dimer"):
        return _exact_full(c, probs[0], more)
    if c["kind"] == "displaced":
        p = probs[0]
        pairs, scale = more.moved
        p.v.view(len(p.pairs), -1)[torch.from_numpy(pairs).to(p.v.device)] *= torch.from_numpy(scale).to(p.v.device)[:, None]
    got = [_exact_doubles(p, tol) for p in probs]
    if not fp64:
        for g in got:
            del g["sweeps"]
    if c["kind"] == "served":
        return got
    if c["kind"] != "batch":
        return got[0]
    out = {k: np.concatenate([g[k] for g in got]) for k in ("e_m2", "de_m2", "e_d2", "t")}
    out["clusters"] = np.array([g["total"] for g in got])
    out["total"] = out["clusters"].sum(0)
    if fp64:
        out["sweeps"] = max(g["sweeps"] for g in got)
    return out

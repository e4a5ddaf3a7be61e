"""Cases that stand for the work users of this framework have it do.

Each case is a graph, a method and a number of queries per call.  The graph is
resident (loaded once, as a serving program keeps it); what is new from pass
to pass is the queries.  Graphs: R-MAT power-law graphs of the benchmark's
parameters (any vertex count), and the two synthetic inputs of the paper, the
3D grid and randLocal.  Methods: PR-Nibble on the plain path (one query after
another, the optimized rule or the original one, a single seed or a seed set),
HK-PR, Nibble, the batch engine with dense and with compact state, and its
submit/progress loop.
"""
from __future__ import annotations

import ctypes
import functools
import math

import numpy as np
import torch

import paper_1604_07515_amd as plc

DEV = "cuda" if torch.cuda.is_available() else "cpu"
RMAT = (0.57, 0.19, 0.19, 0.05)
RANGE = 30_000  # randLocal's largest id offset


# ------------------------------------------------------------------- graphs

def _csr(n, u, v):
    """Simple undirected CSR (sorted rows, no self-loops) of the edges (u, v), on the host."""
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.cat([u * n + v, v * n + u]))
    src = key // n
    off = torch.zeros(n + 1, dtype=torch.int64, device=key.device)
    off[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    return off.cpu().numpy(), (key - src * n).to(torch.int32).cpu().numpy()


@functools.lru_cache(maxsize=None)
def graph(kind, n, ef):
    """Host CSR (off int64, nbr int32) of a case's graph."""
    gen = torch.Generator(device=DEV).manual_seed(1)
    if kind == "rmat":  # ef * n samples over the next power of two, those past n left out
        m = int(ef) * n
        u = torch.zeros(m, dtype=torch.int64, device=DEV)
        v = torch.zeros(m, dtype=torch.int64, device=DEV)
        a, b, c, _ = RMAT
        for _ in range(max(1, (n - 1).bit_length())):
            x = torch.rand(m, generator=gen, device=DEV)
            u = 2 * u + (x >= a + b)
            v = 2 * v + (((x >= a) & (x < a + b)) | (x >= a + b + c))
        keep = (u < n) & (v < n)
        return _csr(n, u[keep], v[keep])
    if kind == "grid":  # n = side^3 torus
        side = round(n ** (1 / 3))
        i = torch.arange(n, device=DEV)
        x, y, z = i % side, (i // side) % side, i // (side * side)
        j = [(x + 1) % side + y * side + z * side * side,
             x + ((y + 1) % side) * side + z * side * side,
             x + y * side + ((z + 1) % side) * side * side]
        return _csr(n, i.repeat(3), torch.cat(j))
    u = torch.arange(n, device=DEV).repeat_interleave(5)  # randLocal
    d = torch.exp(torch.rand(len(u), generator=gen, device=DEV, dtype=torch.float64)
                  * math.log(min(RANGE, n - 1))).to(torch.int64)
    return _csr(n, u, (u + d) % n)


def inputs(case, seed):
    """The queries of a case: seeds, alpha and eps per query."""
    off, _ = graph(case["graph"], case["n"], case["ef"])
    rng = np.random.default_rng(seed)
    deg = np.diff(off)
    k = case["count"]
    if case["by"] == "degree":  # the source of a uniformly drawn arc
        s = np.searchsorted(off, rng.integers(0, off[-1], k), side="right") - 1
    else:
        cand = np.flatnonzero(deg >= (8 if case["by"] == "inside" else 1))
        s = cand[rng.integers(0, len(cand), k)]
    alpha = np.asarray((0.01, 0.05))[rng.integers(0, 2, k)] if case["alpha"] == 0 \
        else np.full(k, float(case["alpha"]))
    lo, hi = math.log10(case["eps"]), math.log10(case["eps_hi"])
    return s.astype(np.int32), alpha, 10.0 ** rng.uniform(lo, hi, k)


# -------------------------------------------------------------------- cases

def case(name, method, graph, n, ef, count=1, by="uniform", alpha=0.01, eps=1e-7, eps_hi=0.0,
         slots=0, N=0, t=0.0):
    c = dict(method=method, graph=graph, n=n, ef=ef, count=count, by=by, alpha=alpha, eps=eps,
             eps_hi=eps_hi or eps, slots=slots, N=N, t=t)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one query on a small graph, residual kept and returned
        case("one_rmat12", "residual", "rmat", 1 << 12, 8, eps=1e-3),
        # an interactive query on an ordinary graph of ragged size: latency counts
        case("one_rmat20", "plain", "rmat", 1_000_003, 16, alpha=0.05, eps=1e-6),
        # the benchmark's headline step: 16 seeds one after another
        case("plain16_rmat22", "plain", "rmat", 1 << 22, 16, count=16),
        # a query that covers the whole component (the benchmark's C1)
        case("saturating_rmat16", "plain", "rmat", 1 << 16, 8, by="inside"),
        # the paper's own two synthetic inputs, many rounds of small frontiers
        case("grid215", "plain", "grid", 215 ** 3, 3),
        case("randlocal_1e7", "plain", "local", 10_000_000, 5),
        # a seed set under the original push rule
        case("set64_orig_rmat18", "set", "rmat", 200_003, 16, count=64, eps=1e-6),
        # the paper's other two diffusions, with the benchmark's parameters
        case("hkpr_rmat22", "hkpr", "rmat", 1 << 22, 16, N=20, t=10.0),
        case("nibble_rmat22", "nibble", "rmat", 1 << 22, 16, eps=1e-8, N=20),
        # the benchmark's batch of 256 with either state layout
        case("batch256_dense", "batch", "rmat", 1 << 22, 16, count=256, alpha=0, eps_hi=1e-5,
             slots=256),
        case("batch256_compact", "compact", "rmat", 1 << 22, 16, count=256, alpha=0, eps_hi=1e-5,
             slots=256),
        # a serving loop at saturation: more queries than slots, compact tables
        case("serve512_rmat20", "serve", "rmat", 1 << 20, 16, count=512, by="degree",
             eps_hi=1e-4, slots=128),
    ]


def draw(rng):
    def log(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    m = rng.choice(("plain", "plain", "residual", "set", "hkpr", "nibble", "batch", "compact",
                    "serve"))
    g = rng.choice(("rmat", "rmat", "rmat", "grid", "local"))
    alpha = rng.choice((0.01, 0.05))
    if m in ("batch", "compact", "serve"):
        n = int(log(1 << 14, 1 << 21))
        k = int(log(8, 256))
        return case(None, m, "rmat", n, rng.randint(8, 16), count=k, by="degree", alpha=0,
                    eps=log(1e-7, 1e-6), eps_hi=1e-4, slots=min(256, max(4, k // rng.randint(1, 3))))
    n = int(log(1 << 12, 1 << 21))
    if g == "grid":
        n = max(9, round(n ** (1 / 3))) ** 3
    ef = rng.randint(8, 16) if g == "rmat" else 3 if g == "grid" else 5
    if m == "hkpr":
        return case(None, m, g, n, ef, eps=log(1e-7, 1e-5), N=rng.randint(5, 30), t=rng.uniform(3, 10))
    if m == "nibble":
        return case(None, m, g, n, ef, eps=log(1e-8, 1e-6), N=rng.randint(5, 30))
    k = 1 if m == "residual" else int(log(1, 16)) if m == "plain" else int(log(2, 200))
    return case(None, m, g, n, ef, count=k, alpha=alpha, eps=log(1e-7, 1e-5))


class State:
    """A context with the case's graph loaded, its queries, and buffers for their results."""

    def __init__(self, case, seed):
        self.case = case
        self.method = case["method"]
        off, nbr = graph(case["graph"], case["n"], case["ef"])
        n, arcs = len(off) - 1, len(nbr)
        self.n = n
        self.seeds, self.alpha, self.eps = inputs(case, seed)
        compact = self.method in ("compact", "serve")
        arena = plc.plain_arena_bytes(n, arcs) + (512 << 20)
        if case["slots"]:
            arena += plc.batch_arena_bytes(n, arcs, case["slots"], compact=compact,
                                           table_bytes=(8 << 30) if compact else 0)
        self.ctx = plc.Context(arena, compact=compact)
        self.g = self.ctx.load_graph(off, nbr)
        if case["slots"]:
            self.ctx.batch_reserve(self.g, case["slots"])
        # where the library copies supports and p, and where the program keeps them (by id)
        k = room(case)
        self.pin_ids = torch.zeros(k, dtype=torch.int32, pin_memory=True)
        self.pin_p = torch.zeros(k, dtype=torch.float64, pin_memory=True)
        self.h_ids, self.h_p = self.pin_ids.numpy(), self.pin_p.numpy()
        where = "cpu" if on_host(case) else DEV
        self.ids = torch.zeros(k, dtype=torch.int64, device=where)
        self.p = torch.zeros(k, dtype=torch.float64, device=where)
        if self.method in ("residual", "set"):
            self.r_ids, self.r = np.zeros(n, np.int32), np.zeros(n)

    def __del__(self):
        if getattr(self, "ctx", None):
            self.ctx.close()


def room(case):
    """Vertices the result buffers of a call hold."""
    return min(case["count"] * case["n"], 4_000_000)


def on_host(case):
    """Small results stay on the host; large ones go back to the GPU, where a program that joins
    them with per-vertex data keeps them."""
    return case["method"] in ("residual", "set", "nibble") or \
        (case["method"] == "plain" and case["count"] == 1 and case["graph"] != "local")


def prepare(case, seed):
    return State(case, seed)


COUNTS = ["status", "rounds", "pushes", "edges", "support", "kstar", "cut", "vol"]


def _infos(s, qids):
    """Result records of finished queries."""
    rec = (plc.plc_result_info * len(qids))()
    for i, q in enumerate(qids):
        s.ctx.lib.plc_result_info_get(s.ctx.handle, q, ctypes.byref(rec[i]))
    return np.frombuffer(rec, dtype=np.dtype(plc.plc_result_info))


def _fetch(s, qids, rec, at=0):
    """Copy supports and p of the queries end to end into the pinned buffers from position at on,
    and release the results."""
    size = rec["support"]
    end = at + int(size.sum())
    if end > len(s.h_ids):
        raise MemoryError("result buffers")
    first = at + np.cumsum(size) - size
    args = [np.asarray(qids, np.uint64), (s.h_ids.ctypes.data + 4 * first).astype(np.uint64),
            (s.h_p.ctypes.data + 8 * first).astype(np.uint64)]
    if s.method in ("residual", "set"):
        s.got = np.empty(int(rec["r_nnz"][0]), np.int32), np.empty(int(rec["r_nnz"][0]))
        args += [np.array([x.ctypes.data], np.uint64) for x in s.got]
    ptr = [x.ctypes.data for x in args] + [None] * (5 - len(args))
    rc = s.ctx.lib.plc_result_copy_many(s.ctx.handle, len(qids), *ptr)
    if rc != plc.PLC_OK:
        raise plc.PlcError(rc, "plc_result_copy_many")
    for q in qids:
        s.ctx.release(q)
    return end


def _keep(s, which, size):
    """The fetched supports and p into the state's own vectors, query by query in id order
    (ids of query q counted from q * n on)."""
    end = int(size.sum())
    if s.ids.device.type == "cpu":
        order = np.argsort(s.h_ids[:end])
        s.ids.numpy()[:end] = s.h_ids[:end][order]
        s.p.numpy()[:end] = s.h_p[:end][order]
    else:
        key = s.pin_ids[:end].to(DEV, non_blocking=True).long()
        if len(size) > 1:
            size_d = torch.from_numpy(size.astype(np.int64)).to(DEV)
            base = torch.from_numpy(np.asarray(which, np.int64) * s.n).to(DEV)
            key += torch.repeat_interleave(base, size_d, output_size=end)
        s.ids[:end], order = torch.sort(key)
        s.p[:end] = s.pin_p[:end].to(DEV, non_blocking=True)[order]
    return s.ids, s.p


def _told(rec):
    return np.stack([rec[k].astype(np.int64) for k in COUNTS], 1), rec["phi"].copy()


def run(s):
    ctx, g, m, c = s.ctx, s.g, s.method, s.case
    if m == "serve":  # every query waits in the queue; each step's results leave at once
        qids = ctx.submit(g, s.seeds, s.alpha, s.eps, flags=plc.PLC_QF_NO_RESIDUAL)
        index = {q: i for i, q in enumerate(qids)}
        which, recs, at, left = [], [], 0, 1
        while left:
            done = []
            left = ctx.progress(g, done)
            if done:
                recs.append(_infos(s, done))
                at = _fetch(s, done, recs[-1], at)
                which += [index[q] for q in done]
        rec = np.concatenate(recs)
        back = np.argsort(which)
        return _told(rec[back]) + _keep(s, which, rec["support"])
    if m in ("batch", "compact"):
        qids, _ = ctx.run_batched(g, s.seeds, s.alpha, s.eps, flags=plc.PLC_QF_NO_RESIDUAL)
    elif m == "hkpr":
        qids = [ctx.run_hkpr(g, int(s.seeds[0]), c["N"], float(s.eps[0]), c["t"])[0]]
    elif m == "nibble":
        qids = [ctx.run_nibble(g, int(s.seeds[0]), float(s.eps[0]), c["N"])[0]]
    elif m == "set":
        qids = [ctx.run_set(g, s.seeds, float(s.alpha[0]), float(s.eps[0]), plc.PLC_RULE_ORIG)[0]]
    else:
        qids, _ = ctx.run(g, s.seeds.tolist(), float(s.alpha[0]), float(s.eps[0]),
                          flags=0 if m == "residual" else plc.PLC_QF_NO_RESIDUAL)
    rec = _infos(s, qids)
    _fetch(s, qids, rec)
    out = _told(rec) + _keep(s, range(len(qids)), rec["support"])
    if m in ("residual", "set"):
        order = np.argsort(s.got[0])
        s.r_ids[:len(order)], s.r[:len(order)] = s.got[0][order], s.got[1][order]
        out += (s.r_ids, s.r)
    return out


# ------------------------------------------------- the same in plain float64

class Plain:
    """Dense float64 evaluation of the methods on one graph, straight from their definitions."""

    def __init__(self, off, nbr):
        self.off = torch.from_numpy(off).to(DEV)
        self.nbr = torch.from_numpy(nbr).to(DEV)
        self.n = len(off) - 1
        self.deg = torch.diff(self.off).double()
        self.edges = self.pushes = 0

    def arcs(self, F):
        """Neighbour of every arc of the vertices F, and the position in F it belongs to."""
        d = self.off[F + 1] - self.off[F]
        own = torch.repeat_interleave(torch.arange(len(F), device=DEV), d)
        first = torch.cumsum(d, 0) - d
        at = torch.arange(len(own), device=DEV) + (self.off[F] - first)[own]
        return self.nbr[at].long(), own

    def push(self, F, coef, into):
        w, own = self.arcs(F)
        self.edges += len(w)
        self.pushes += len(F)
        into.index_add_(0, w, coef[own])
        return torch.unique(w)

    def prnibble(self, seeds, alpha, eps, orig):
        cs, cn, keep = (alpha, (1 - alpha) / 2, (1 - alpha) / 2) if orig else \
            (2 * alpha / (1 + alpha), (1 - alpha) / (1 + alpha), 0.0)
        p = torch.zeros(self.n, dtype=torch.float64, device=DEV)
        r = torch.zeros_like(p)
        F = torch.unique(torch.as_tensor(np.asarray(seeds, np.int64), device=DEV))
        r[F] = 1.0 / len(F)
        while len(F):
            rho = r[F]
            p[F] += cs * rho
            r[F] = keep * rho
            c = torch.unique(torch.cat([self.push(F, cn * rho / self.deg[F], r), F]))
            F = c[r[c] >= eps * self.deg[c]]
        return p, r

    def hkpr(self, x, N, eps, t):
        p = torch.zeros(self.n, dtype=torch.float64, device=DEV)
        r = torch.zeros_like(p)
        r[x] = 1.0
        F = torch.tensor([x], device=DEV)
        for j in range(N):
            if not len(F):
                break
            rho = r[F]
            p[F] += rho
            if j + 1 == N:
                self.push(F, rho / self.deg[F], p)
                break
            k, term, psi = j + 1, 1.0, 1.0
            for i in range(1, N - k + 1):
                term *= t / (k + i)
                psi += term
            r = torch.zeros_like(p)
            c = self.push(F, t * rho / ((j + 1) * self.deg[F]), r)
            F = c[r[c] >= math.exp(-t) * eps * self.deg[c] / (2 * N * psi)]
        return p

    def nibble(self, x, eps, T):
        p = torch.zeros(self.n, dtype=torch.float64, device=DEV)
        p[x] = 1.0
        F = torch.tensor([x], device=DEV)
        for _ in range(T):
            q = torch.zeros_like(p)
            q[F] = p[F] / 2
            c = torch.unique(torch.cat([self.push(F, p[F] / (2 * self.deg[F]), q), F]))
            F = c[q[c] >= eps * self.deg[c]]
            if not len(F):
                break
            p = q
        return p

    def conductance(self, p):
        """The smallest conductance of a prefix of the sweep order."""
        S = torch.nonzero(p).reshape(-1)
        S = S[torch.sort(p[S] / self.deg[S], descending=True, stable=True)[1]]
        rank = torch.full((self.n,), self.n, dtype=torch.int64, device=DEV)
        rank[S] = torch.arange(len(S), device=DEV)
        w, own = self.arcs(S)
        inner = torch.bincount(own[rank[w] < own], minlength=len(S))
        d = (self.off[S + 1] - self.off[S])
        vol = torch.cumsum(d, 0)
        cut = torch.cumsum(d - 2 * inner, 0).double()
        den = torch.minimum(vol, len(self.nbr) - vol)
        return float(torch.where(den > 0, cut / den.clamp(min=1), math.inf).min())


@functools.lru_cache(maxsize=1)
def _plain(kind, n, ef):
    return Plain(*graph(kind, n, ef))


def _evaluate(case, seed):
    """(p, r) of each query of the case, one at a time; r is None where the method has none."""
    G = _plain(case["graph"], case["n"], case["ef"])
    seeds, alpha, eps = inputs(case, seed)
    m = case["method"]
    if m == "hkpr":
        yield G.hkpr(int(seeds[0]), case["N"], float(eps[0]), case["t"]), None
    elif m == "nibble":
        yield G.nibble(int(seeds[0]), float(eps[0]), case["N"]), None
    elif m == "set":
        yield G.prnibble(seeds, float(alpha[0]), float(eps[0]), True)
    else:
        for x, a, e in zip(seeds, alpha, eps):
            yield G.prnibble([x], float(a), float(e), False)


def exact(case, seed):
    G = _plain(case["graph"], case["n"], case["ef"])
    ps, phis, r = [], [], None
    for p, r in _evaluate(case, seed):
        ps.append(p[p != 0])
        phis.append(G.conductance(p))
    ps = torch.cat(ps)
    out = (None, np.array(phis), None, torch.nn.functional.pad(ps, (0, room(case) - len(ps))))
    if case["method"] in ("residual", "set"):
        r = r[r != 0]
        out += (None, torch.nn.functional.pad(r, (0, G.n - len(r))))
    return out


@functools.lru_cache(maxsize=None)
def _work(key):
    """Counted on one set of queries: bytes are the rows of the pushed vertices (8 B of offset
    and 4 B per arc) and the support with p (12 B per vertex), each once; flops are an addition
    and a comparison per pushed arc and four per push."""
    case = dict(key)
    G = _plain(case["graph"], case["n"], case["ef"])
    G.edges = G.pushes = 0
    moved = 0
    for p, _ in _evaluate(case, 0):
        S = torch.nonzero(p).reshape(-1)
        moved += 20 * len(S) + 4 * int(G.deg[S].sum())
    return moved, 2 * G.edges + 4 * G.pushes


def work(case):
    b, f = _work(tuple(sorted((k, v) for k, v in case.items() if k != "name")))
    return {"bytes": b, "flops": f}

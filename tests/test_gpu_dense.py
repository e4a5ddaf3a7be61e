"""GPU parity of the dense rounds (plain path): every row sums its neighbours'
coefficients and takes its next self step in the same launch.

Sizes where the form can go wrong: rows at the length where they are cut into
pieces (2048 arcs) and one past it, a row of many pieces, blocks that end at
256 rows, isolated vertices, the way into the form and back to the frontier
list, the round limit inside it, the beta variant (which lists the next
frontier), and HK-PR levels.  All against the CPU oracle, or the same query
through the atomic scatter; tolerance and near-tie handling as for every other
form (only the order of a row's additions differs).
"""
import numpy as np
import pytest

import oracle
import synth
from parity import check_hkpr, check_query, check_same

pytestmark = pytest.mark.gpu

OPT, ORIG = 0, 1


def joined_stars(sizes, gap):
    """Stars of the given leaf counts, their hubs on a path, `gap` isolated
    vertices behind each."""
    edges, hubs, v = [], [], 0
    for k in sizes:
        hubs.append(v)
        edges += [(v, v + 1 + i) for i in range(k)]
        v += 1 + k + gap
    edges += list(zip(hubs, hubs[1:]))
    return synth.from_edges(v, edges, "stars")


GRAPHS = {
    # hub degrees 2047, 2048, 2049, 4097 and 10001 (the path's edges included)
    "stars": lambda: joined_stars([2046, 2046, 2047, 4095, 10000], 300),
    "rmat13": lambda: synth.rmat(13, 12, seed=4),
    "path600": lambda: synth.path(600),
    "k300": lambda: synth.complete(300),
    # large enough that a shrinking frontier goes back to the list
    "rmat17": lambda: synth.rmat(17, 16, seed=3),
}
_host = {}


@pytest.fixture(scope="module")
def plc():
    import paper_1604_07515_amd as plc
    return plc


def graph(name):
    if name not in _host:
        _host[name] = GRAPHS[name]()
    return _host[name]


def context(plc, g, **kw):
    return plc.Context(arena_bytes=plc.plain_arena_bytes(g.n, g.arcs) + (64 << 20), **kw)


@pytest.mark.parametrize("bin_min_edges", (0, 1, 20000))
@pytest.mark.parametrize("gname,rule,alpha,eps", [
    ("stars", OPT, 0.2, 1e-7), ("stars", ORIG, 0.3, 1e-7), ("rmat13", OPT, 0.01, 1e-7),
    ("rmat13", ORIG, 0.05, 1e-6), ("k300", OPT, 0.05, 1e-6), ("path600", OPT, 0.05, 1e-8)])
def test_dense_parity(plc, gname, rule, alpha, eps, bin_min_edges):
    g = graph(gname)
    seeds = [0, int(np.argmin(np.where(g.deg > 0, g.deg, 1 << 30)))]
    with context(plc, g, bin_min_edges=bin_min_edges) as c:
        hg = c.load_graph(g.off, g.nbr, validate=True)
        for _ in range(2):  # the second pass queues what the first one learned
            ids, infos = c.run(hg, seeds, alpha, eps, rule)
            for qid, s in zip(ids, seeds):
                check_query(g, c.result(qid, release=True), s, alpha, eps, rule)


def test_dense_and_back(plc):
    """The default threshold on a graph of 4 M arcs: the large rounds are
    dense, the rounds before and after them are not."""
    g = graph("rmat17")
    with context(plc, g) as c, context(plc, g, bin_min_edges=-1) as ca:
        hg, ha = c.load_graph(g.off, g.nbr), ca.load_graph(g.off, g.nbr)
        for rule, alpha, eps in ((OPT, 0.05, 1e-6), (ORIG, 0.1, 1e-6)):
            ids, infos = c.run(hg, [0, 5, 77], alpha, eps, rule)
            ref, _ = ca.run(ha, [0, 5, 77], alpha, eps, rule)
            for qid, q2, s in zip(ids, ref, (0, 5, 77)):
                res = c.result(qid, release=True)
                check_same(g, res, ca.result(q2, release=True))
                check_query(g, res, s, alpha, eps, rule)


@pytest.mark.parametrize("rule,alpha", [(OPT, 0.01), (ORIG, 0.05)])
def test_round_limit_inside(plc, rule, alpha):
    g = graph("rmat13")
    for rounds in (3, 7, 8):
        with context(plc, g, max_rounds=rounds) as c, \
                context(plc, g, max_rounds=rounds, bin_min_edges=-1) as ca:
            out = []
            for x in (c, ca):
                hg = x.load_graph(g.off, g.nbr)
                ids, infos = x.run(hg, [1], alpha, 1e-7, rule, check=False)
                assert infos[0]["status"] == plc.PLC_E_LIMIT and infos[0]["rounds"] == rounds
                out.append(x.result(ids[0], release=True))
            check_same(g, *out)


def test_beta_lists_the_frontier(plc):
    """beta below 1 ranks the next frontier, so a dense round lists it; the
    exact PPR mass and the termination hold whatever ties do."""
    g = graph("rmat13")
    with context(plc, g, bin_min_edges=1) as c:
        hg = c.load_graph(g.off, g.nbr)
        for rule in (OPT, ORIG):
            qid, info = c.run_beta(hg, 1, 0.05, 1e-6, 0.9, rule)
            res = c.result(qid, release=True)
            p, r = res.dense_p(g.n), res.dense_r(g.n)
            assert abs(p.sum() + r.sum() - 1.0) < 1e-12
            assert np.all((r < 1e-6 * g.deg) | (r == 0))
        # and a plain query afterwards finds the arrays clean
        ids, _ = c.run(hg, [1], 0.05, 1e-6)
        check_query(g, c.result(ids[0], release=True), 1, 0.05, 1e-6, OPT)


@pytest.mark.parametrize("gname,seed,N,eps,t", [
    ("stars", 1, 1, 1e-6, 2.0), ("stars", 1, 2, 1e-6, 2.0), ("stars", 0, 9, 1e-7, 4.0),
    ("rmat13", 3, 12, 1e-6, 5.0), ("rmat17", 3, 15, 1e-6, 6.0), ("rmat17", 9, 15, 1e-4, 4.0)])
@pytest.mark.parametrize("bin_min_edges", (0, 600000))
def test_hkpr_levels(plc, gname, seed, N, eps, t, bin_min_edges):
    g = graph(gname)
    with context(plc, g, bin_min_edges=bin_min_edges) as c:
        hg = c.load_graph(g.off, g.nbr)
        want = oracle.hkpr(g.off, g.nbr, seed, N, eps, t)
        for _ in range(2):
            qid, info = c.run_hkpr(hg, seed, N, eps, t)
            check_hkpr(g, c.result(qid, release=True), want)
        # the residual arrays are clean again
        ids, _ = c.run(hg, [seed], 0.05, 1e-5)
        check_query(g, c.result(ids[0], release=True), seed, 0.05, 1e-5, OPT)

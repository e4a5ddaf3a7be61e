"""Queries whose rounds go into the dense form, back to the list form and in
again, at rounds of either parity, under the default rule (a graph of more than
2^20 arcs) and under a fixed threshold; and the beta variant's dense rounds,
whose next frontier is listed.  All against the CPU oracle.

Which rounds are dense follows from their edges, which are simulated here:
those of at least (2m - 2^20) / 4 edges with the default, of at least half the
arcs with a fixed threshold.  The library counts them where they also have the
threshold's edges and half the arcs (pull_rounds).
"""
import numpy as np
import pytest

import oracle
import synth
from parity import check_query

OPT, ORIG = 0, 1
LOOP_EDGES, LOOP_VERTICES = 4096, 1024  # a self launch runs rounds up to this by itself

GRAPHS = {"rmat12": lambda: synth.rmat(12, 12, seed=4), "rmat13": lambda: synth.rmat(13, 12, seed=4),
          "rmat15": lambda: synth.rmat(15, 32, seed=3), "rmat16": lambda: synth.rmat(16, 16, seed=3),
          "rmat16d": lambda: synth.rmat(16, 24, seed=3),
          "er300": lambda: synth.erdos_renyi(300, 0.03, 7)}
_host = {}

# graph, seed, alpha, eps, rule, bin_min_edges
CASES = [("rmat15", 5, 0.02, 3e-7, OPT, 0), ("rmat15", 5, 0.02, 3e-7, ORIG, 0),
         ("rmat16", 5, 0.02, 3e-7, OPT, 0), ("rmat16d", 5, 0.1, 1e-7, ORIG, 0),
         ("rmat16d", 5, 0.2, 1e-8, OPT, 0), ("rmat12", 1, 0.01, 1e-5, OPT, 5000),
         ("rmat12", 1, 0.01, 1e-5, ORIG, 5000), ("rmat13", 1, 0.05, 3e-6, OPT, 5000),
         ("rmat13", 1, 0.05, 3e-6, ORIG, 5000)]


def graph(name):
    if name not in _host:
        _host[name] = GRAPHS[name]()
    return _host[name]


def round_edges(g, x, alpha, eps, rule):
    """(vertices, edges) of every round's frontier."""
    deg = np.asarray(g.deg, np.float64)
    src = np.repeat(np.arange(g.n), np.diff(g.off))
    cn, keep = ((1 - alpha) / (1 + alpha), 0.0) if rule == OPT else ((1 - alpha) / 2,) * 2
    r = np.zeros(g.n)
    r[x] = 1.0
    F = np.zeros(g.n, bool)
    F[x] = True
    out = []
    while F.any():
        out.append((int(F.sum()), int(deg[F].sum())))
        coef = np.where(F, cn * r / np.maximum(deg, 1), 0.0)
        r = np.where(F, keep * r, r) + np.bincount(g.nbr, weights=coef[src], minlength=g.n)
        F = (r >= eps * deg) & (deg > 0)
    return out


def forms(g, emin, rounds):
    """Per round: 'd' dense, 'w' wide enough for the scatter launch, 'l' a self launch's own."""
    def form(nf, E):
        wide = nf > LOOP_VERTICES or E > LOOP_EDGES
        dense = g.arcs <= (1 << 20) + 4 * E if emin == 0 else E >= emin and 2 * E >= g.arcs
        return "d" if dense and wide else "w" if wide else "l"
    return "".join(form(*x) for x in rounds)


def test_cases_leave_and_return():
    """The cases go dense, list and dense again, entering at even and at odd rounds."""
    entries = {0: set(), 5000: set()}
    for name, x, alpha, eps, rule, emin in CASES:
        s = forms(graph(name), emin, round_edges(graph(name), x, alpha, eps, rule))
        first = s.index("d")
        assert "wd" in s[first:], s
        entries[emin] |= {(first + i + 1) % 2 for i in range(len(s[first:]) - 1)
                          if s[first + i] != "d" and s[first + i + 1] == "d"}
        if emin == 0:
            assert graph(name).arcs > 1 << 20
    assert entries == {0: {0, 1}, 5000: {0, 1}}


@pytest.mark.gpu
@pytest.mark.parametrize("name,x,alpha,eps,rule,emin", CASES)
def test_dense_list_dense(name, x, alpha, eps, rule, emin):
    import paper_1604_07515_amd as plc
    g = graph(name)
    rounds = round_edges(g, x, alpha, eps, rule)
    want = oracle.prnibble(g.off, g.nbr, x, alpha, eps, rule)
    assert want.min_rel_gap > 1e-10
    assert (len(rounds), sum(e for _, e in rounds)) == (want.rounds, want.edges)
    least = emin or 524288
    wide = [e for _, e in rounds if e >= least]
    half = [e for e in wide if 2 * e >= g.arcs]
    assert half
    with plc.Context(plc.plain_arena_bytes(g.n, g.arcs) + (64 << 20), bin_min_edges=emin) as c:
        hg = c.load_graph(g.off, g.nbr)
        for _ in range(3):  # later passes queue what the earlier ones needed
            ids, infos = c.run(hg, [x], alpha, eps, rule)
            check_query(g, c.result(ids[0], release=True), x, alpha, eps, rule, orc=want)
            assert infos[0]["pull_rounds"] == len(half)
            assert (infos[0]["bin_rounds"], infos[0]["bin_edges"]) == (len(wide), sum(wide))


@pytest.mark.gpu
@pytest.mark.parametrize("rule,beta,eps", [(OPT, 0.9, 1e-4), (OPT, 0.9, 1e-6), (ORIG, 0.9, 3e-5),
                                           (ORIG, 0.9, 1e-6)])
def test_beta_dense_values(rule, beta, eps):
    """Rounds that push at least half the arcs, where the ranking never ties: p, r, the
    counters and the sweep are the oracle's."""
    import paper_1604_07515_amd as plc
    g = graph("er300")
    x = int(np.argmax(g.deg))
    want = oracle.prnibble_beta(g.off, g.nbr, x, 0.01, eps, beta, rule)
    assert min(want.min_rel_gap, want.min_sel_gap) > 1e-10
    with plc.Context(64 << 20, bin_min_edges=1) as c:
        hg = c.load_graph(g.off, g.nbr)
        qid, info = c.run_beta(hg, x, 0.01, eps, beta, rule)
        out = check_query(g, c.result(qid, release=True), x, 0.01, eps, rule, orc=want)
        assert not out["tie_push"] and info["pull_rounds"] > 0

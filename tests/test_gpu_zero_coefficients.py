"""HK-PR levels whose coefficients underflow to 0: the vertices still belong to
the level's frontier, and their additions of 0 touch nothing (in the list form
the touched list holds n vertices, and the level makes more additions), also
when the level goes back from the dense to the list form (which lists the
frontier from the coefficient array).

With t = 1e-98 a level-k residual is about 1e-98^k / (k! d^k): level 3 is
still a normal number, level 4 is 0.  eps is put between the level-3 ratios
r/d, so that level 2 covers more than half of the arcs (dense) and level 3
less (list), with a 0 coefficient at every vertex of it.
"""
import numpy as np
import pytest

import oracle
import synth
from parity import check_hkpr

T, N = 1e-98, 8


def case(name):
    """Graph, seed and an eps that lets less than half of the arcs' volume pass at level 3."""
    g = {"rmat9": lambda: synth.rmat(9, 8, seed=2), "rmat12": lambda: synth.rmat(12, 12, seed=5)}[name]()
    deg = np.asarray(g.deg, np.float64)
    src = np.repeat(np.arange(g.n), np.diff(g.off))
    x = int(np.argmax(deg))
    level = {0: np.zeros(g.n)}
    level[0][x] = 1.0
    for k in range(3):
        coef = np.where(deg > 0, (T * level[k]) / ((k + 1) * np.maximum(deg, 1)), 0.0)
        level[k + 1] = np.bincount(g.nbr, weights=coef[src], minlength=g.n)
    on = level[3] > 0
    ratio = level[3][on] / deg[on]
    order = np.argsort(-ratio)
    part = np.searchsorted(np.cumsum(deg[on][order]), g.arcs / 4)
    psi = 1.0  # 1 + t/k + ... = 1 in double precision
    eps = float(np.sqrt(ratio[order][part]) * np.sqrt(ratio[order][part + 1])) * 2 * N * psi
    return g, x, eps, level


@pytest.mark.parametrize("name", ("rmat9", "rmat12"))
def test_case(name):
    """The cases are what the docstring says."""
    g, x, eps, level = case(name)
    deg = np.asarray(g.deg, np.float64)
    act = [np.sum(deg[(level[k] > 0) & (level[k] >= eps * deg / (2 * N))]) for k in (2, 3)]
    assert act[0] >= (g.arcs + 1) // 2 > act[1] > 0
    on = level[3] > 0
    assert level[3][on].min() > 1e-307 and np.all(T * level[3][on] == 0.0)
    assert act[1] > g.n  # the additions of 0
    assert oracle.hkpr(g.off, g.nbr, x, N, eps, T).levels == 4


@pytest.mark.gpu
@pytest.mark.parametrize("bin_min_edges", (-1, 1, 0))
@pytest.mark.parametrize("name", ("rmat9", "rmat12"))
def test_zero_coefficients(name, bin_min_edges):
    import paper_1604_07515_amd as plc
    g, x, eps, _ = case(name)
    want = oracle.hkpr(g.off, g.nbr, x, N, eps, T)
    with plc.Context(plc.plain_arena_bytes(g.n, g.arcs) + (64 << 20),
                     bin_min_edges=bin_min_edges) as c:
        hg = c.load_graph(g.off, g.nbr)
        for _ in range(2):
            qid, info = c.run_hkpr(hg, x, N, eps, T)
            check_hkpr(g, c.result(qid, release=True), want)

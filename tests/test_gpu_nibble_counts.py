"""Nibble steps report how many of them were binned (plc_result_info.bin_rounds
and bin_edges): those of at least the threshold's edges, all of them with a
threshold of 1, none with the binned form off.  A graph's first query queues the
second pass behind every step."""
import numpy as np
import pytest

import oracle
import synth
from parity import check_nibble

pytestmark = pytest.mark.gpu


def step_edges(g, x, eps, T):
    """Edges of every step's frontier."""
    deg = np.asarray(g.deg, np.float64)
    src = np.repeat(np.arange(g.n), np.diff(g.off))
    p = np.zeros(g.n)
    p[x] = 1.0
    F = np.zeros(g.n, bool)
    F[x] = True
    out = []
    for _ in range(T):
        if not F.any():
            break
        out.append(int(deg[F].sum()))
        on = np.where(F, p, 0.0)
        half = on / (2.0 * np.maximum(deg, 1))
        p = on / 2.0 + np.bincount(g.nbr, weights=half[src], minlength=g.n)
        F = (p >= eps * deg) & (p > 0)
    return out


@pytest.mark.parametrize("emin", (1, 3000, -1))
@pytest.mark.parametrize("gname,eps,T", [("rmat14", 1e-6, 15), ("torus12", 1e-5, 20)])
def test_nibble_counts(gname, eps, T, emin):
    import paper_1604_07515_amd as plc
    g = {"rmat14": lambda: synth.rmat(14, 8, seed=2), "torus12": lambda: synth.torus3d(12)}[gname]()
    x = int(np.flatnonzero(g.deg == g.deg[g.deg > 0].min())[0])
    want = oracle.nibble(g.off, g.nbr, x, eps, T)
    edges = step_edges(g, x, eps, T)
    assert want.min_rel_gap > 1e-10 and sum(edges) == want.edges and len(edges) == want.iterations
    wide = [e for e in edges if 0 < emin <= e]
    if emin == 3000:
        assert 0 < len(wide) < len(edges)
    with plc.Context(1 << 30, bin_min_edges=emin) as c:
        hg = c.load_graph(g.off, g.nbr)
        qid, info = c.run_nibble(hg, x, eps, T)
        check_nibble(g, c.result(qid, release=True), want)
        assert (info["bin_rounds"], info["bin_edges"]) == (len(wide), sum(wide))
        assert info["pull_rounds"] == 0

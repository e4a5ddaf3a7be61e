"""GPU parity of Nibble steps in the destination-binned form (entries' own
halves added first, the neighbours' contributions by bin afterwards) against
the oracle, with thresholds that bin every step or only the wider ones, and
queries that follow one whose first binned step was earlier or later (the
steps before it are then queued without the second pass)."""
import numpy as np
import pytest

import oracle
import synth
from parity import check_nibble

pytestmark = pytest.mark.gpu

GRAPHS = {"rmat16": lambda: synth.rmat(16, 8, seed=2), "torus12": lambda: synth.torus3d(12),
          "star300": lambda: synth.star(300), "path3": lambda: synth.path(3)}


@pytest.mark.parametrize("emin", (1, 3000))
@pytest.mark.parametrize("gname", sorted(GRAPHS))
def test_nibble_binned(gname, emin):
    import paper_1604_07515_amd as plc
    g = GRAPHS[gname]()
    hub, low = int(np.argmax(g.deg)), int(np.flatnonzero(g.deg == g.deg[g.deg > 0].min())[0])
    with plc.Context(1 << 30, bin_min_edges=emin) as c:
        hg = c.load_graph(g.off, g.nbr)
        for x, eps, T in ((low, 1e-4, 12), (hub, 1e-7, 20), (low, 1e-300, 6), (hub, 1e-3, 20),
                          (low, 1e-7, 20), (hub, 1e-300, 5)):
            print("case", gname, emin, x, eps, T, flush=True)
            qid, _ = c.run_nibble(hg, x, eps, T)
            check_nibble(g, c.result(qid, release=True), oracle.nibble(g.off, g.nbr, x, eps, T))

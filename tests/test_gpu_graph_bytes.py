"""plc_graph_info.bytes is what the graph takes of the arena."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bin_min_edges", (0, -1))
def test_graph_bytes(bin_min_edges):
    import paper_1604_07515_amd as plc
    for g in (synth.path(2), synth.star(5000), synth.rmat(14, 12, seed=1)):
        with plc.Context(plc.plain_arena_bytes(g.n, g.arcs), bin_min_edges=bin_min_edges) as c:
            before = c.arena_free()[0]
            hg = c.load_graph(g.off, g.nbr)
            assert hg.info()["bytes"] == before - c.arena_free()[0]
            hg.free()
            assert c.arena_free()[0] == before

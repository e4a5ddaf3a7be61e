"""Results copied ahead of the read-back that tells their sizes: queries whose
support or residual outgrows the block that the queries before them suggest,
with and without residuals, alone and as the last of several, and from an
arena whose free blocks are too small; the arena holds afterwards what the
results need and nothing more."""
import numpy as np
import pytest

import synth
from parity import check_query

pytestmark = pytest.mark.gpu

NO_R = 1  # PLC_QF_NO_RESIDUAL


def test_sizes_grow_and_shrink():
    import paper_1604_07515_amd as plc
    assert plc.PLC_QF_NO_RESIDUAL == NO_R
    g = synth.rmat(13, 8, seed=4)
    seeds = [int(v) for v in synth.uniform_seeds(g, 3, seed=2)]
    with plc.Context(plc.plain_arena_bytes(g.n, g.arcs) + (64 << 20)) as c:
        hg = c.load_graph(g.off, g.nbr)
        start = c.arena_free()
        held = []
        for k, (eps, flags, many) in enumerate(
                ((1e-3, 0, 1), (1e-3, 0, 1), (1e-6, 0, 1), (1e-6, 0, 3), (1e-3, NO_R, 1),
                 (1e-7, NO_R, 1), (1e-7, 0, 1), (1e-4, 0, 3), (1e-7, NO_R, 3), (1e-2, 0, 1))):
            s = seeds[:many]
            ids, infos = c.run(hg, s, 0.05, eps, flags=flags)
            for x, q, info in zip(s, ids, infos):
                res = c.result(q)
                if flags == 0:
                    check_query(g, res, x, 0.05, eps, 0)
                else:
                    ref = c.run(hg, [x], 0.05, eps)[0][0]
                    full = c.result(ref, release=True)
                    assert np.allclose(full.dense_p(g.n), res.dense_p(g.n), rtol=1e-12, atol=0)
                    assert len(full.sweep_ids) == len(res.sweep_ids) == info["support"]
                    assert len(res.r_ids) == 0
            held += ids
            while len(held) > 4:  # holes of several sizes in the arena
                c.release(held.pop(len(held) // 2 if k % 2 else 0))
            N = [c.result_info(q) for q in held]
            need = sum(-(-(4 * i["support"]) // 256) * 256 + -(-(8 * i["support"]) // 256) * 256
                       + (0 if i["flags"] & NO_R else -(-(4 * i["r_nnz"]) // 256) * 256
                          + -(-(8 * i["r_nnz"]) // 256) * 256) for i in N)
            assert start[0] - c.arena_free()[0] == need
        for q in held:
            c.release(q)
        assert c.arena_free() == start

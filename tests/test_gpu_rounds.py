"""Frontier sizes where the plain path's list rounds change hands: the self
launch's own loop takes up to 1024 vertices and 4096 edges, a larger frontier
that the loop leaves goes through the scatter launch, the entry scan gives one
block per workgroup up to 256 blocks of 1024 and a ticket above.

A star pushed from its hub with eps between cn^2/k and cn/k takes exactly two
rounds: the hub, then all k leaves, each with the same residual cn/k (one
addition, so p is exact), after which the hub's own residual (k equal
additions, up to 2 (k - 1) u relative) stays below its threshold.  The sweep
then orders 1 + k vertices, k of them exactly tied.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", (3, 255, 256, 257, 1023, 1024, 1025, 4095, 4096, 4097, 65536,
                               262143, 262144, 262145))
def test_star_frontiers(k):
    import paper_1604_07515_amd as plc
    n = k + 1
    off = np.concatenate([[0], np.arange(k, 2 * k + 1)]).astype(np.int64)
    nbr = np.concatenate([np.arange(1, n), np.zeros(k)]).astype(np.int32)
    g = synth.Graph(off, nbr, "star")
    alpha = 0.3
    cs, cn = 2.0 * alpha / (1.0 + alpha), (1.0 - alpha) / (1.0 + alpha)
    leaf = cn / float(k)
    with plc.Context(plc.plain_arena_bytes(n, g.arcs) + (64 << 20), bin_min_edges=-1) as c:
        hg = c.load_graph(off, nbr)
        for _ in range(2):  # the scan sites' two descriptor buffers
            ids, infos = c.run(hg, [0], alpha, 0.4 / k)
            info = infos[0]
            assert (info["rounds"], info["pushes"], info["edges"]) == (2, n, 2 * k)
            assert info["support"] == n and info["r_nnz"] == 1
            res = c.result(ids[0], release=True)
            p, r = res.dense_p(n), res.dense_r(n)
            assert p[0] == cs and np.all(p[1:] == cs * leaf)
            assert abs(r[0] - cn * cn) <= 2 * (k + 4) * 2.0 ** -53 * cn * cn
            # leaves first or the hub first, by p/d; equal ratios by id
            order = np.lexsort((np.arange(n), -(p / g.deg)))
            assert np.array_equal(res.sweep_ids, order)
            assert np.array_equal(res.sweep_p, p[order])

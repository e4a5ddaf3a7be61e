"""Batched sweeps at the sizes where the sort changes hands: tiles of 1024
elements, merge groups of 4096, and segments of at most 32,768 elements (one
larger segment takes the whole sweep to the general sort).

Hub-and-leaves graphs side by side, leaf i with 2 - i % 3 leaves of its own.
Pushed from a hub with eps between cn^2/(2k) and cn/(3k) (k leaves; at alpha
0.5 cn = 1/3), a query takes exactly two rounds, the hub and its k leaves: a
leaf's residual is one addition, so p is exact, its own leaves stay below the
threshold, and the sweep orders k + 1 vertices in three classes of p/d, equal
ones by id.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = (2, 3, 1023, 1024, 1025, 4096, 4097, 8193, 32768)


def hubs(sizes):
    deg, nbr, at = [], [], []
    base = 0
    for n_elem in sizes:
        k = n_elem - 1
        extra = 2 - np.arange(k) % 3
        leaf = base + 1 + np.arange(k)
        first = base + 1 + k + np.cumsum(extra) - extra
        owner = np.repeat(leaf, extra)
        rows = np.stack([np.full(k, base), first, first + 1], 1)
        keep = np.arange(3)[None, :] <= extra[:, None]
        at.append(base)
        deg += [[k], extra + 1, np.ones(len(owner), np.int64)]
        nbr += [leaf, rows[keep], owner]
        base += 1 + k + len(owner)
    deg = np.concatenate(deg)
    off = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    return off, np.concatenate(nbr).astype(np.int32), deg, at


@pytest.mark.parametrize("compact", (False, True))
@pytest.mark.parametrize("sizes", (SIZES, SIZES + (32769,)))
def test_segments(sizes, compact):
    import paper_1604_07515_amd as plc
    off, nbr, deg, at = hubs(sizes)
    n, arcs = len(deg), len(nbr)
    alpha = 0.5
    cs, cn = 2.0 * alpha / (1.0 + alpha), (1.0 - alpha) / (1.0 + alpha)
    arena = plc.plain_arena_bytes(n, arcs) + (256 << 20) + plc.batch_arena_bytes(
        n, arcs, len(sizes), compact=compact, table_bytes=(1 << 30) if compact else 0)
    with plc.Context(arena, compact=compact) as c:
        hg = c.load_graph(off, nbr)
        assert c.batch_reserve(hg, len(sizes)) == len(sizes)
        eps = np.array([0.09 / (m - 1) for m in sizes])
        for _ in range(2):
            ids, infos = c.run_batched(hg, np.array(at), np.full(len(sizes), alpha), eps)
            for q, (hub, m) in enumerate(zip(at, sizes)):
                k = m - 1
                info = infos[q]
                assert (info["rounds"], info["pushes"], info["support"]) == (2, m, m)
                res = c.result(ids[q], release=True)
                v = hub + np.arange(m)
                p = np.concatenate([[cs], np.full(k, cs * (cn / float(k)))])
                order = np.lexsort((v, -(p / deg[v])))
                assert np.array_equal(res.sweep_ids, v[order])
                assert np.array_equal(res.sweep_p, p[order])
                # the sweep's cut and volume at k*: only the tree edges between members are inside
                s = set(v[order][: info["kstar"]].tolist())
                vol = int(sum(deg[x] for x in s))
                inside = sum(1 for x in s if x != hub) if hub in s else 0
                assert info["vol"] == vol and info["cut"] == vol - 2 * inside

"""Queries on two contexts at once, each on a stream and a host thread of its
own: the launches of both share the chip, and every result is the one the
context gives alone (against the oracle).  Frontiers of several scan blocks, so
that the workgroups of the scans wait for one another."""
import threading

import pytest

import oracle
import synth
from parity import check_query

pytestmark = pytest.mark.gpu

ALPHA, EPS, RULES = 0.02, 1e-7, (0, 1)


def test_two_contexts_at_once():
    import torch
    import paper_1604_07515_amd as plc
    graphs = [synth.rmat(16, 8, seed=11), synth.torus3d(40)]
    seeds = [[int(s) for s in synth.uniform_seeds(g, 3, seed=4)] for g in graphs]
    want = [{(s, r): oracle.prnibble(g.off, g.nbr, s, ALPHA, EPS, r) for s in ss for r in RULES}
            for g, ss in zip(graphs, seeds)]
    ctxs = [plc.Context(plc.plain_arena_bytes(g.n, g.arcs) + (256 << 20),
                        stream=torch.cuda.Stream(), bin_min_edges=-1) for g in graphs]
    handles = [c.load_graph(g.off, g.nbr) for c, g in zip(ctxs, graphs)]
    batched = [c.batch_reserve(h, 3) for c, h in zip(ctxs, handles)]
    got, errors = [[], []], []

    def work(i):
        try:
            for rule in RULES:
                for _ in range(6):
                    for run in (ctxs[i].run, ctxs[i].run_batched):
                        ids, _ = run(handles[i], seeds[i], ALPHA, EPS, rule)
                        got[i] += [(s, rule, ctxs[i].result(q, release=True))
                                   for s, q in zip(seeds[i], ids)]
        except Exception as e:  # (shown by the main thread)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    assert batched == [3, 3]
    for i, g in enumerate(graphs):
        assert len(got[i]) == 2 * 2 * 6 * 3
        for s, rule, res in got[i]:
            check_query(g, res, s, ALPHA, EPS, rule, orc=want[i][s, rule])
    for c in ctxs:
        c.close()

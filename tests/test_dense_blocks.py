"""The dense rounds' blocks of rows (C++ check, CPU), and the arena bytes that
plain_arena_bytes counts for them and leaves for results."""
import os
import subprocess

import numpy as np
import pytest

import synth
import paper_1604_07515_amd as plc

HERE = os.path.dirname(os.path.abspath(__file__))


def test_dense_blocks(tmp_path):
    exe = str(tmp_path / "dense_blocks_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-o", exe,
                           os.path.join(HERE, "dense_blocks_check.cpp")])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr
    lines = out.stdout.split("\n")
    assert "blocks ok" in lines
    for line in lines[:lines.index("blocks ok")]:
        n, arcs, most = map(int, line.split())
        assert plc.dense_table_bytes(n, arcs) >= 32 * most + 12 * (arcs // 2049 + 1) + 64 * 128


@pytest.mark.parametrize("n,arcs", [(1 << 22, 128 << 20), (1536 * 4096, 2100 << 20),
                                    (1536 * 4096, 40 << 30), (100_000, 9 << 30), (2, 2)])
def test_plain_arena_bytes(n, arcs):
    """What plc_graph_load takes, array by array, and 64 MiB: the largest graphs with bins, where
    the blocks of rows are many."""
    vertex = 8 + 16 + 8 + 2 * 4 + 3 * 8 + 2 * 4 + 2 * 16 + 4 + 8 + 4 + 8 + 4 + 4 + 8 + 4 + 8 + 2 * 4
    chunks = (min(arcs, 1 << 23) + 2047) // 2048
    need = (vertex + 16) * n + 4 * arcs + 4 * (arcs // 1024 + 2) + 72 * (n // 1024 + 2)
    need += 4 * (n // 64 + 1) + chunks * 8 * 2048
    need += chunks * 4 * (n // 4096 + 1)  # the bins that their width alone makes
    blocks = n // 256 + 2 * arcs // 2048  # typical for rows of one length
    assert plc.plain_arena_bytes(n, arcs) >= need + 32 * blocks + (64 << 20)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ("path2", "k2050", "k1025", "rmat16", "torus40"))
def test_room_for_results(name):
    """A graph loaded into an arena of plain_arena_bytes leaves the 64 MiB for results."""
    g = {"path2": lambda: synth.path(2), "rmat16": lambda: synth.rmat(16, 16, seed=1),
         "torus40": lambda: synth.torus3d(40)}.get(name)
    if g:
        g = g()
        n, off, nbr = g.n, g.off, g.nbr
    else:  # complete graphs: rows of 2049 arcs (two pieces each), blocks of one row
        n = int(name[1:])
        off = np.arange(n + 1, dtype=np.int64) * (n - 1)
        nbr = np.arange(n - 1, dtype=np.int32)[None, :] + \
            (np.arange(n - 1)[None, :] >= np.arange(n)[:, None]).astype(np.int32)
        nbr = np.ascontiguousarray(nbr.reshape(-1), dtype=np.int32)
    with plc.Context(plc.plain_arena_bytes(n, len(nbr))) as c:
        c.load_graph(off, nbr)
        assert c.arena_free()[0] >= 64 << 20

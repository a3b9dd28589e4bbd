"""Merging a batch into a resident state's edge and type lists: removed edges at
the borders of the 64-edge words and the workgroups that find them, whole rows,
first and last edges, and graphs whose length is or misses a multiple of 64."""

import numpy as np
import pytest

from paper_2111_12493_amd import graphgen as gg

from test_gpu_incremental import Session

pytestmark = pytest.mark.gpu


def graph(m, n, seed):
    # distinct triples: edge e is (row, e % 3, a target of its own)
    rng = np.random.default_rng(seed)
    src = np.sort(rng.integers(0, n, m))
    return gg.from_edges(n, src, np.arange(m) % n, np.arange(m) % 3, types=[[int(t)] for t in rng.integers(0, 4, n)])


def edge(g, e):
    v = int(np.searchsorted(g.row_off, e, side="right") - 1)
    return v, int(g.lab[e]), int(g.tgt[e])


@pytest.mark.parametrize("m", [0, 1, 63, 64, 65, 128, 255, 256, 257, 1023, 1024, 1025, 4096, 4161])
def test_removed_edges_at_word_borders(m):
    n = 40
    g = graph(m, n, m)
    s = Session(g, 3, stop=False)
    at = sorted({e for b in (0, 63, 64, 127, 128, 255, 256, 1023, 1024, m - 65, m - 64, m - 2, m - 1)
                 for e in (b,) if 0 <= e < m})
    ops = [("del_e", *edge(g, e)) for e in at]
    ops += [("add_e", 1, 2, 3), ("mod_v", 2, [9]), ("mod_v", n - 1, [])]
    s.apply(ops, what=("word borders", m))
    s.apply([("add_e", n - 1, 1, 0), ("add_v", [7]), ("add_e", n, 0, 1)], what=("after", m))
    s.apply([("del_v", 0), ("del_v", n - 1)], what=("rows", m))
    s.close()


@pytest.mark.parametrize("hub", [64, 300, 2500])
def test_rows_over_many_words(hub):
    # one row that spans words and workgroups loses every third edge
    n = 60
    src = np.concatenate([np.zeros(5, int), np.full(hub, 1), np.arange(n)])
    tgt = np.concatenate([np.arange(5), np.arange(hub) % n, np.arange(n)[::-1]])
    lab = np.concatenate([np.zeros(5, int), np.arange(hub) // n, np.ones(n, int)])
    g = gg.from_edges(n, src, tgt, lab, types=[[i % 3] for i in range(n)])
    s = Session(g, 2, stop=False)
    s.apply([("del_e", 1, int(e // n), int(e % n)) for e in range(0, hub, 3)], what=("thirds", hub))
    s.apply([("del_v", 5)], what=("a target of the row", hub))
    s.apply([("del_v", 1)], what=("the row", hub))
    s.close()

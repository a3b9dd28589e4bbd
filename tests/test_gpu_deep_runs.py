"""Runs past 256 levels, whose class tests go over from launches of their own to
the next level's launch: fixpoints and caps around the change, with and without
the stop test, previous-level edges, hubs and solo vertices beside a path, every
level kept (a resident state), batches, and both ends of the queueing option."""

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2111_12493_amd import binding
from paper_2111_12493_amd import graphgen as gg

from gpu_util import assert_same

pytestmark = pytest.mark.gpu
UNB = binding.K_UNBOUNDED
DEEP = 256


def path_and_rows(length, seed=1):
    """A path of `length` edges behind a hub, a solo vertex and a tile's vertex,
    beside a sparse rest: the path changes at every level."""
    rng = np.random.default_rng(seed)
    n = length + 900
    deg = [2300, 700, 60]
    src = np.concatenate([np.repeat(np.arange(3), deg), np.arange(3, length + 3), rng.integers(length + 4, n, 1500)])
    tgt = np.concatenate([rng.integers(3, n, sum(deg)), np.arange(4, length + 4), rng.integers(length + 4, n, 1500)])
    lab = np.concatenate([rng.integers(0, 3, sum(deg)), np.zeros(length, int), rng.integers(0, 3, 1500)])
    return gg.from_edges(n, src, tgt, lab, types=[[0]] * (length + 4) + [[int(t)] for t in rng.integers(1, 4, n - length - 4)])


def run(c, g, k_max=UNB, stop=True, prev=False, timed=0):
    c.set_option("time_launches", timed)
    r = binding.summarize(c, binding.DeviceGraph(g), k_max=k_max, stop_at_fixpoint=stop, prev_level_edges=prev)
    d = r.to_dict()
    d["timed"], d["split"], d["launches"] = r.n_timed_launches, r.n_split_launches, r.n_iter_launches
    r.free()
    return d


@pytest.mark.parametrize("ppm", [0, 100])
@pytest.mark.parametrize("chunk_max", [1, 32])
@pytest.mark.parametrize("length", [DEEP - 3, DEEP - 2, DEEP - 1, DEEP, DEEP + 1, DEEP + 2, 700])
def test_fixpoints_around_the_change(length, chunk_max, ppm):
    c = binding.Context(0)
    c.set_option("chunk_max", chunk_max)
    c.set_option("tail_split_ppm", ppm)
    g = path_and_rows(length)
    got, ref = run(c, g, timed=1), orc.summarize(g, g.n + 2, True)
    assert length <= ref["k_done"] <= length + 4
    assert_same(got, ref, (length, chunk_max, ppm))
    # hashing launches: one level past the last where the test looks two back
    k, lag2 = ref["k_done"], ppm == 0 or ref["k_done"] >= DEEP
    assert got["timed"] == k + (1 if lag2 else 0)
    assert got["split"] == (0 if ppm == 0 else min(got["launches"], DEEP))
    c.close()


@pytest.mark.parametrize("ppm", [0, 100])
@pytest.mark.parametrize("stop", [False, True])
@pytest.mark.parametrize("k_max", [DEEP - 2, DEEP - 1, DEEP, DEEP + 1, DEEP + 2, DEEP + 3, 400])
def test_caps_around_the_change(k_max, stop, ppm):
    c = binding.Context(0)
    c.set_option("tail_split_ppm", ppm)
    g = path_and_rows(DEEP + 60)
    assert_same(run(c, g, k_max, stop), orc.summarize(g, k_max, stop), (k_max, stop, ppm))
    ref = orc.summarize(g, k_max, stop, prev_level_edges=True)
    assert_same(run(c, g, k_max, stop, prev=True), ref, ("prev", k_max, stop, ppm))
    c.close()


@pytest.mark.parametrize("ppm", [0, 100])
@pytest.mark.parametrize("small_edges", [0, 10 ** 9])
def test_batches_past_the_change(small_edges, ppm):
    c = binding.Context(0)
    c.set_option("batch_small_edges", small_edges)
    c.set_option("tail_split_ppm", ppm)
    graphs = [path_and_rows(n, n) for n in (3, DEEP - 2, DEEP - 1, DEEP, DEEP + 1, 500)] + \
             [gg.chain(n) for n in (5, DEEP - 1, DEEP, DEEP + 1, DEEP + 2, 1100)]
    for k_max, stop in ((UNB, True), (DEEP, False), (DEEP + 1, True), (DEEP + 2, False)):
        rs = binding.batch_summarize(c, [binding.DeviceGraph(g) for g in graphs], k_max=k_max, stop_at_fixpoint=stop)
        for i, (g, r) in enumerate(zip(graphs, rs)):
            ref = orc.summarize(g, k_max if k_max != UNB else g.n + 2, stop)
            assert_same(r.to_dict(), ref, (i, k_max, stop, small_edges, ppm))
            r.free()
    c.close()


@pytest.mark.parametrize("k_max", [DEEP - 1, DEEP, DEEP + 1, DEEP + 4])
def test_states_of_many_levels(k_max):
    c = binding.Context(0)
    g = path_and_rows(DEEP + 30)
    s = binding.State(c, binding.DeviceGraph(g), k_max)
    assert_same(s.result.to_dict(), orc.summarize(g, k_max, False), k_max)
    # an update reads every level that was kept
    r = s.apply(binding.UpdateBatch([("add_e", 5, 1, DEEP + 40)]))
    after = s.graph()
    assert_same(r.to_dict(), orc.summarize(after, k_max, False), ("update", k_max))
    r.free()
    s.free()
    c.close()

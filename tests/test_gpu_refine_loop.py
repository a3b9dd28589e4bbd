"""The refinement loop's queueing: runs longer than the ring of report words,
every number of launches queued ahead, with and without the stop test seeing
the level just hashed, capped and uncapped, and founders spread over more
waves than there are counters."""

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2111_12493_amd import binding
from paper_2111_12493_amd import graphgen as gg

from gpu_util import assert_same

pytestmark = pytest.mark.gpu
UNB = binding.K_UNBOUNDED


def run(c, g, k_max, stop):
    r = binding.summarize(c, binding.DeviceGraph(g), k_max=k_max, stop_at_fixpoint=stop)
    d = r.to_dict()
    d["launches"], d["split"] = r.n_iter_launches, r.n_split_launches
    r.free()
    return d


@pytest.mark.parametrize("ppm", [0, 100])
@pytest.mark.parametrize("chunk_max", [1, 2, 3, 4, 64])
def test_levels_past_the_report_ring(chunk_max, ppm):
    c = binding.Context(0)
    c.set_option("chunk_max", chunk_max)
    c.set_option("tail_split_ppm", ppm)
    g = gg.append_chains(gg.rmat_graph(9, 1 << 11, n_types=8, n_labels=4, seed=3), 2, 150, type_id=8)
    for k_max, stop in ((UNB, True), (63, False), (64, True), (65, False), (0, False), (1, True)):
        got = run(c, g, k_max, stop)
        assert_same(got, orc.summarize(g, g.n + 2 if k_max == UNB else k_max, stop), (chunk_max, ppm, k_max, stop))
        # launches that hash or return at once: never more than are queued ahead
        assert got["launches"] <= got["k_done"] + (2 if ppm == 0 else 1) + min(chunk_max, 4)
        assert got["split"] == (got["launches"] if ppm else 0)
    c.close()


@pytest.mark.parametrize("n", [1, 255, 1024, 1025, 66000])
def test_founders_of_every_wave(n):
    # level 0 founds a class per vertex; level 1 splits pairs apart
    g = gg.from_edges(n, np.arange(n // 2), (np.arange(n // 2) * 7 + 1) % n, np.zeros(n // 2, dtype=np.int64),
                      types=[[i // 2] for i in range(n)])
    c = binding.Context(0)
    assert_same(run(c, g, UNB, True), orc.summarize(g, g.n + 2, True), n)
    c.close()

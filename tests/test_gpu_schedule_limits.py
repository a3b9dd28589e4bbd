"""The schedule's limits as the library's header states them: tiles of 64
vertices and 512 edges, solo vertices up to 2,048 edges, hubs above, their
chunks of 1,536 edges and the 512 chunk runs that a bucket stages at a time, and
hub lists longer than the 4,096 that come back with the counts.  The limits are
read from the header, so the cases move with them."""

import os
import re

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2111_12493_amd import binding
from paper_2111_12493_amd import graphgen as gg

from gpu_util import assert_same, check

pytestmark = pytest.mark.gpu

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2111_12493_amd", "csrc")


def _limits():
    names = {}
    for f in ("bsim_internal.h", "bsim_iter.hip", "bsim_stage.hip"):
        with open(os.path.join(CSRC, f)) as h:
            for n, v in re.findall(r"constexpr \w+ (k\w+) = ([^;]+);", h.read()):
                try:
                    names[n] = int(eval(v, {"__builtins__": {}}, names))
                except Exception:
                    pass
    return names


LIM = _limits()
V, E, SOLO = LIM["kTileMaxVerts"], LIM["kTileMaxEdges"], LIM["kSoloMaxEdges"]
CHUNK, RUNS, COPY, GROUP = LIM["kChunkEdges"], LIM["kMaxHubRuns"], LIM["kStageHubs"], LIM["kStageVerts"]


def graph_of_degrees(deg, seed, u16=False, n_labels=40):
    rng = np.random.default_rng(seed)
    deg = np.asarray(deg, dtype=np.int64)
    n, m = deg.size, int(deg.sum())
    g = gg.from_edges(n, np.repeat(np.arange(n), deg), rng.integers(0, n, size=m), rng.integers(0, n_labels, size=m),
                      types=[[int(t)] for t in rng.integers(0, 6, size=n)])
    return gg.with_u16_labels(g) if u16 else g


def test_the_limits_were_read():
    assert (V, E, SOLO, CHUNK, RUNS, COPY, GROUP) == (64, 512, 2048, 1536, 512, 4096, 2048)


DEGREES = {
    "tiles ended by their vertices": [1] * (V - 1) + [E] + [1] * V + [E] + [1] * (V + 1) + [0] * 9 + [2] * (4 * V + 1),
    "tiles ended by their edges": [E // 2 - 1, E // 2, E // 2 + 1, 1, E, 1, E - 1, 1, 1, E - 1, 2, E] * 12,
    "tile and solo vertices": [E - 1, E, E + 1, 3, E + 1, E + 1, E, 1, 0, E + 2] * 7,
    "solo vertices and hubs": [SOLO - 1, 5, SOLO, SOLO + 1, 0, SOLO + 1, SOLO, 2, 2 * CHUNK, 2 * CHUNK + 1],
    "last vertex of a workgroup": [1] * (GROUP - 1) + [E + 1] + [1] * (GROUP - 1) + [SOLO + 1] + [1] * (GROUP - 1) + [E],
    "only solo vertices": [E + 1, SOLO, E + 1] * 5,
    "only hubs": [SOLO + 1, 3 * CHUNK, 3 * CHUNK + 1],
}


@pytest.mark.parametrize("u16", [False, True])
@pytest.mark.parametrize("name", sorted(DEGREES))
def test_degrees_at_the_limits(name, u16):
    check(graph_of_degrees(DEGREES[name], len(name), u16), 4, stop=False, what=name)


@pytest.mark.parametrize("more", [0, 4])
def test_hub_lists_around_one_copy(more):
    # (the second copy of the hub list is made only past kStageHubs hubs)
    deg = np.full(COPY + more + 200, 2, dtype=np.int64)
    deg[20:20 + COPY + more] = SOLO + 1
    deg[20] = 9000
    deg[20 + COPY + more - 1] = 5000
    check(graph_of_degrees(deg, 9, u16=True), 1, stop=False, what=more)


@pytest.mark.parametrize("edges", [RUNS * CHUNK, RUNS * CHUNK + 1, 900_000])
def test_hubs_of_more_chunks_than_are_staged_at_once(edges):
    g = graph_of_degrees([edges, SOLO + 1] + [3] * 20000, 8)
    check(g, 3, stop=False, what=edges)


def test_runs_staged_again_with_few_slots():
    # a hub whose buckets are re-split while their runs come in several batches
    c = binding.Context(0)
    c.set_option("hub_table_slots", 1024)
    g = graph_of_degrees([RUNS * CHUNK + 1] + [2] * 30000, 3, n_labels=7)
    r = binding.summarize(c, binding.DeviceGraph(g), k_max=2, stop_at_fixpoint=False)
    assert_same(r.to_dict(), orc.summarize(g, 2, False), "few slots")
    r.free()
    c.close()

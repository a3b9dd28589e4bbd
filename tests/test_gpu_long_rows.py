"""Rows longer than a tile in the passes over all edges (edge sources of a view,
values of the summary edges): hubs cut at the borders of their chunks of 1,536
edges beside solo vertices, in every direction and under a label set."""

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2111_12493_amd import binding
from paper_2111_12493_amd import graphgen as gg

from gpu_util import assert_same, ctx

pytestmark = pytest.mark.gpu

DEGREES = [
    [2049],
    [0, 3071, 3072, 3073, 2048, 4608, 1, 4607, 4609, 513],
    [100001, 3, 2048, 0, 2049],
]


def graph(deg, u16):
    rng = np.random.default_rng(len(deg))
    n = len(deg) + 300
    src = np.concatenate([np.repeat(np.arange(len(deg)), deg), rng.integers(0, n, 500)])
    tgt = rng.integers(0, n, src.size)
    lab = rng.integers(0, 50, src.size)
    g = gg.from_edges(n, src, tgt, lab, types=[[int(t)] for t in rng.integers(0, 4, n)], n_labels=50)
    return gg.with_u16_labels(g) if u16 else g


@pytest.mark.parametrize("labels", [None, range(0, 50, 2)])
@pytest.mark.parametrize("direction", ["out", "in", "both"])
@pytest.mark.parametrize("u16", [False, True])
@pytest.mark.parametrize("deg", DEGREES, ids=len)
def test_chunks_of_long_rows(deg, u16, direction, labels):
    g = graph(deg, u16)
    r = binding.summarize(ctx(), binding.DeviceGraph(g), k_max=2, stop_at_fixpoint=False, direction=direction,
                          labels=labels)
    ref = orc.summarize_ext(g, 2, False, direction=direction, labels=labels)
    assert_same(r.to_dict(), ref, (deg, direction, labels))
    r.free()

"""Reversed edge lists at their edges: targets far apart (gaps longer than one
edge fills in), all edges into one vertex, no kept edge, and vertices and
labels too wide for a packed sort key; bit-exact against the oracle."""

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2111_12493_amd import binding
from paper_2111_12493_amd import graphgen as gg

from gpu_util import assert_same, ctx

pytestmark = pytest.mark.gpu


def graph(n, src, dst, lab, seed):
    rng = np.random.default_rng(seed)
    types = rng.integers(0, 3, size=n).astype(np.uint32)
    return gg.from_edges(n, src, dst, lab, typ_off=np.arange(n + 1, dtype=np.uint64), typ=types)


def cases():
    rng = np.random.default_rng(5)
    out = {}
    m = 3000
    for name, n, dst in (("gaps of 64 and 65", 2000, np.array([0, 64, 129, 195, 1999])),
                         ("one target first", 70000, np.array([0])),
                         ("one target last", 70000, np.array([69999])),
                         ("every vertex", 700, np.arange(700))):
        out[name] = graph(n, rng.integers(0, n, m), rng.choice(dst, m), rng.integers(0, 9, m), 1)
    # 21 + 21 bits of vertices and 24 of label pass 64
    n = (1 << 20) + 5
    out["wide labels"] = graph(n, rng.integers(0, n, m), rng.integers(n - 300, n, m),
                               rng.choice([0, 7, (1 << 23) + 1, (1 << 23) + 9], m), 2)
    return out


CASES = cases()


@pytest.mark.parametrize("labels", [None, [0, 2, 7], [1 << 20]])
@pytest.mark.parametrize("direction", ["in", "both"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_reversed_rows(name, direction, labels):
    g = CASES[name]
    ref = orc.summarize_ext(g, 3, False, direction=direction, labels=labels)
    r = binding.summarize(ctx(), binding.DeviceGraph(g), k_max=3, stop_at_fixpoint=False, direction=direction,
                          labels=labels)
    assert_same(r.to_dict(), ref, (name, direction, labels))
    r.free()

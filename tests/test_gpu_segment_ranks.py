"""Short summary-edge segments, whose values are ranked by counting: lengths on
both sides of the wave and of the longest that is counted, tiles of as many
segments as fit, repeated values, and values of 32 and of more bits."""

import numpy as np
import pytest

from paper_2111_12493_amd import graphgen as gg

from gpu_util import check

pytestmark = pytest.mark.gpu

LEAVES = 700


def segments(sizes, distinct, max_label, seed):
    # one vertex and one block per size; `distinct` bounds the labels drawn, so
    # values repeat; the leaves are blocks of their own
    rng = np.random.default_rng(seed)
    k = len(sizes)
    sizes = np.asarray(sizes)
    m = int(sizes.sum())
    src = np.repeat(LEAVES + np.arange(k), sizes)
    dst = rng.integers(0, LEAVES, m) if distinct > 1 else np.zeros(m, dtype=np.int64)
    lab = rng.integers(0, distinct, m) * (max_label // max(distinct - 1, 1))
    types = [[i] for i in range(LEAVES + k)]
    return gg.from_edges(LEAVES + k, src, dst, lab, types=types)


SIZES = {
    "pairs": [2] * 700,
    "with singles": [1, 2, 1, 3, 1, 1] * 120,
    "around a wave": [63, 64, 65, 1, 62, 64, 66] * 9,
    "around the longest": [127, 128, 129, 2, 128, 128, 3] * 6,
    "one at a tile's end": [2] * 127 + [1] + [128] + [2] * 100 + [256] + [5] * 60,
    "mixed": list(range(2, 140)) * 2,
}


@pytest.mark.parametrize("max_label", [7, (1 << 22) - 1, (1 << 24) - 1])
@pytest.mark.parametrize("distinct", [1, 2, 8])
@pytest.mark.parametrize("name", sorted(SIZES))
def test_ranked_segments(name, distinct, max_label):
    g = segments(SIZES[name], distinct, max_label, len(name) + distinct)
    check(g, 1, stop=False, what=(name, distinct, max_label))

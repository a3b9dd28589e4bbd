"""Segments of more than 16,384 values, gathered in runs of 4,096 for one global
sort: runs that end inside, at and past a segment's last value."""

import numpy as np
import pytest

from paper_2111_12493_amd import graphgen as gg

from gpu_util import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[16385], [16385, 16385], [20480, 20480, 3], [16385, 24576, 40961, 16384, 16386],
                                   [70000, 1, 16385]])
@pytest.mark.parametrize("max_label", [5, (1 << 24) - 1])
def test_runs_over_segment_borders(sizes, max_label):
    rng = np.random.default_rng(sum(sizes))
    leaves = 9000
    n, m = leaves + len(sizes), sum(sizes)
    g = gg.from_edges(n, np.repeat(leaves + np.arange(len(sizes)), sizes), rng.integers(0, leaves, m),
                      rng.integers(0, 6, m) * (max_label // 5), types=[[i] for i in range(n)])
    check(g, 1, stop=False, what=(sizes, max_label))

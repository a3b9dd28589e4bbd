"""Longer summary-edge segments at the limits of their classes (128, 512, 4,096
and 16,384 values), with values that spread over the buckets, that lie close
together beside one far off (a bucket too long to count in), and that repeat
(dropped before the buckets are counted again)."""

import numpy as np
import pytest

from paper_2111_12493_amd import graphgen as gg

from gpu_util import check

pytestmark = pytest.mark.gpu

LEAVES = 6000
SIZES = [128, 129, 130, 255, 256, 257, 511, 512, 513, 514, 1024, 1025, 4095, 4096, 4097, 16384, 16385]


def segments(sizes, kind, max_label, seed):
    rng = np.random.default_rng(seed)
    src, dst, lab = [], [], []
    for i, s in enumerate(sizes):
        src.append(np.full(s, LEAVES + i))
        if kind == "spread":
            d, l = rng.integers(0, LEAVES, s), rng.integers(0, max_label + 1, s)
        elif kind == "close":
            d, l = rng.integers(0, 900, s), np.zeros(s, dtype=np.int64)
            l[s // 3] = max_label
        elif kind == "two values":
            d, l = rng.integers(0, 2, s) * (LEAVES - 1), np.zeros(s, dtype=np.int64)
        elif kind == "repeated":
            d, l = rng.integers(0, 40, s) * 149, rng.integers(0, 2, s) * max_label
        else:  # one value, and one that differs
            d, l = np.full(s, 17), np.zeros(s, dtype=np.int64)
            d[s - 1] = 18 if kind == "one off" else 17
        dst.append(d)
        lab.append(l)
    n = LEAVES + len(sizes)
    return gg.from_edges(n, np.concatenate(src), np.concatenate(dst), np.concatenate(lab),
                         types=[[i] for i in range(n)])


@pytest.mark.parametrize("max_label", [1, 60, (1 << 24) - 1])
@pytest.mark.parametrize("kind", ["spread", "close", "two values", "repeated", "one value", "one off"])
def test_class_limits(kind, max_label):
    check(segments(SIZES, kind, max_label, len(kind)), 1, stop=False, what=(kind, max_label))


@pytest.mark.parametrize("size", [129, 500, 513, 4000])
def test_lists_shorter_than_their_grids(size):
    # too few edges for the host to wait for the lists' lengths
    check(segments([size, 5, 129, 600], "repeated", 3, size), 1, stop=False, what=size)


@pytest.mark.parametrize("more", [-1, 0, 1])
def test_wave_segments_on_their_own(more):
    # 4,096 segments of the wave class and one less or more, beside longer ones
    check(segments([129] * (4096 + more) + [600, 2000], "spread", 5, 7 + more), 1, stop=False, what=more)

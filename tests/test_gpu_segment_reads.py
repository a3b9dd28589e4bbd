"""Summary-edge segments around the rule that sends them to counting or to radix
passes: buckets of one length throughout, below, at and above 24 reads per value
and pass, of one repeated value or of neighbouring ones, with values that differ
in one to four bytes, and one long bucket beside short ones."""

import numpy as np
import pytest

from paper_2111_12493_amd import graphgen as gg

from gpu_util import check

pytestmark = pytest.mark.gpu

LEAVES = 40000
SIZES = [129, 200, 511, 512, 513, 1000, 2047, 4095, 4096]


def segments(length, stride, repeated, labels):
    src, dst, lab = [], [], []
    for i, s in enumerate(SIZES):
        j = np.arange(s)
        bucket = j // length if length else np.where(j < s // 3, 0, j)
        d = bucket * stride + (0 if repeated else j % max(length, 1))
        src.append(np.full(s, LEAVES + i))
        dst.append(d % LEAVES)
        lab.append((bucket % 2) * labels)
    order = np.random.default_rng(length).permutation(sum(SIZES))
    src, dst, lab = (np.concatenate(x)[order] for x in (src, dst, lab))
    n = LEAVES + len(SIZES)
    return gg.from_edges(n, src, dst, lab, types=[[i] for i in range(n)])


@pytest.mark.parametrize("labels", [0, 1, (1 << 24) - 1])
@pytest.mark.parametrize("repeated", [True, False])
@pytest.mark.parametrize("stride", [1, 999])
@pytest.mark.parametrize("length", [0, 1, 24, 25, 48, 49, 73, 97, 600])
def test_around_the_rule(length, stride, repeated, labels):
    check(segments(length, stride, repeated, labels), 0, stop=False, what=(length, stride, repeated, labels))

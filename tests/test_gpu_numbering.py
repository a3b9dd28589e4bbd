"""Block numbering and summary-edge size classes at their edges: workgroups of
2,048 vertices, 64-vertex words, classes whose smallest vertex is not their
representative, more classes in a wave than are grouped, scans of one launch
and of three, and more medium and large segments than one launch holds
workgroups for; bit-exact against the oracle."""

import numpy as np
import pytest

from gpu_util import check
from paper_2111_12493_amd import binding
from paper_2111_12493_amd import graphgen as gg

pytestmark = pytest.mark.gpu


def typed(n, of, src=(), dst=(), lab=(), alive=None):
    return gg.from_edges(n, src, dst, lab, typ_off=np.arange(n + 1, dtype=np.uint64),
                         typ=np.asarray(of, dtype=np.uint32), alive=alive)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 2047, 2048, 2049, 16384 * 2048 // 512, 70001])
@pytest.mark.parametrize("classes", [1, 5, 1 << 30])
def test_numbering(n, classes):
    rng = np.random.default_rng(n)
    of = rng.integers(0, min(classes, max(1, n // 2)), n)
    alive = (rng.random(n) < 0.9).astype(np.uint8) if n % 2 else None
    check(typed(n, of, alive=alive), 1, stop=False, what=(n, classes))


def test_late_members_of_large_classes():
    # level 1 splits every class by whether the one edge is there: the
    # members below the founder of the new class come in any order
    n = 200000
    rng = np.random.default_rng(3)
    src = np.flatnonzero(rng.random(n) < 0.4)
    check(typed(n, np.zeros(n), src, np.full(src.size, 7), np.zeros(src.size, dtype=np.int64)), 2, stop=False)


def test_no_edges_many_vertices():
    check(typed(40000, np.arange(40000) % 17), binding.K_UNBOUNDED)


@pytest.mark.parametrize("size,count", [(257, 9000), (4097, 1100), (16385, 3)])
def test_more_segments_than_workgroups(size, count):
    # `count` vertices, each a class of its own, of `size` distinct edges
    n = count + size
    src = np.repeat(np.arange(count), size)
    dst = count + np.tile(np.arange(size), count)
    g = typed(n, np.concatenate([np.arange(count), np.full(size, count)]), src, dst, np.tile(np.arange(size) % 3, count))
    check(g, 0, stop=False, what=(size, count))

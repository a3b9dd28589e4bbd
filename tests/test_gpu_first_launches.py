"""What the first launches of a call leave for the later ones: the status that
staging puts together from what each workgroup saw, the label salts written
beside the type hashes (also when there are more labels than vertices), and
the counters cleared while the classes are numbered."""

import numpy as np
import pytest

from paper_2111_12493_amd import binding
from paper_2111_12493_amd import graphgen as gg

from gpu_util import check, ctx

pytestmark = pytest.mark.gpu


def graph(n, deg, n_labels, seed, max_label=None):
    rng = np.random.default_rng(seed)
    m = n * deg
    lab = rng.integers(0, n_labels, size=m)
    if max_label is not None and m:
        lab[m // 2] = max_label
    types = [list(rng.integers(0, 5, size=int(c))) for c in rng.integers(0, 3, size=n)]
    return gg.from_edges(n, np.repeat(np.arange(n), deg), rng.integers(0, max(n, 1), size=m), lab, types=types)


@pytest.mark.parametrize("max_label", [0, 255, 256, 65536, (1 << 24) - 1])
def test_more_labels_than_vertices(max_label):
    check(graph(7, 5, max_label + 1, max_label, max_label), 3, stop=False, what=max_label)


@pytest.mark.parametrize("n,deg", [(1, 0), (300, 0), (1, 1), (2049, 3)])
@pytest.mark.parametrize("repeat", [2])
def test_counters_start_at_zero(n, deg, repeat):
    # the second call finds the first one's counts in the work memory
    g = graph(n, deg, 9, n + deg)
    for _ in range(repeat):
        check(g, 4, what=(n, deg))


@pytest.mark.parametrize("v", [0, 2047, 2048, 6000])
def test_most_types_of_any_workgroup(v):
    n = 6001
    types = [[1]] * n
    types[v] = list(range(4097))
    g = gg.from_edges(n, np.arange(n), np.arange(n)[::-1].copy(), np.zeros(n, dtype=np.int64), types=types)
    with pytest.raises(binding.BsimError) as e:
        binding.summarize(ctx(), binding.DeviceGraph(g), k_max=1)
    assert e.value.status == binding.E_UNSUPPORTED
    types[v] = list(range(4096))
    check(gg.from_edges(n, np.arange(n), np.arange(n)[::-1].copy(), np.zeros(n, dtype=np.int64), types=types), 2)


@pytest.mark.parametrize("e", [0, 1, 4097, -1])
def test_largest_label_of_any_workgroup(e):
    g = graph(3000, 3, 4, 5)
    g.lab[e] = 1 << 24
    with pytest.raises(binding.BsimError) as err:
        binding.summarize(ctx(), binding.DeviceGraph(g), k_max=1)
    assert err.value.status == binding.E_UNSUPPORTED

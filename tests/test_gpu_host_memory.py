"""Host results lie in ordinary memory: a forked process reads them, any number
may be kept, and they come through the context's pinned staging whole at the
limits of its small block and of its two halves, also from several threads."""

import ctypes
import os
import threading

import numpy as np
import pytest

from paper_2111_12493_amd import binding
from paper_2111_12493_amd import graphgen as gg

pytestmark = pytest.mark.gpu
FIELDS = sorted(binding.Result.FIELDS)


def graph(n, m=0):
    rng = np.random.default_rng(n)
    return binding.DeviceGraph(gg.from_edges(n, rng.integers(0, n, m), rng.integers(0, n, m), rng.integers(0, 9, m)))


def summarize(c, g, host=True):
    return binding.summarize(c, g, k_max=2, stop_at_fixpoint=False, result_on_host=host)


def arrays(r):
    return {f: r.fetch(f) for f in FIELDS}


def same(a, b):
    return all(np.array_equal(a[f], b[f]) for f in FIELDS)


def mapping_flags(address):
    inside = False
    with open("/proc/self/smaps") as f:
        for line in f:
            w = line.split()
            if "-" in w[0] and not w[0].endswith(":"):
                lo, hi = (int(x, 16) for x in w[0].split("-"))
                inside = lo <= address < hi
            elif inside and w[0] == "VmFlags:":
                return w[1:]
    return None


@pytest.mark.parametrize("n", [500, 700_000])
def test_a_forked_process_reads_them(n):
    c = binding.Context(0)
    r = summarize(c, graph(n, 3 * n))
    ref = arrays(r)
    for f in FIELDS:
        flags = mapping_flags(ctypes.cast(getattr(r.ptr.contents, f), ctypes.c_void_p).value)
        assert flags and "dc" not in flags and "io" not in flags, (f, flags)   # inherited, not a device's
    pid = os.fork()
    if pid == 0:
        ok = False
        try:
            ok = same(arrays(r), ref)
            r.free()
        finally:
            os._exit(0 if ok else 1)
    assert os.waitpid(pid, 0)[1] == 0
    assert same(arrays(r), ref)
    r.free()
    c.close()


# hashes of 8 n bytes: results of about 1 MiB, then of one, two and three halves of 8 MiB
@pytest.mark.parametrize("n", [1, 87_000, 87_371, 87_376, 87_381, 87_390, 131_072, (1 << 20) - 1, 1 << 20,
                               (1 << 20) + 1, (1 << 21) + 1, 3 << 20])
def test_staging_limits(n):
    c = binding.Context(0)
    g = graph(n)
    dev = summarize(c, g, host=False)
    ref = arrays(dev)
    dev.free()
    for _ in range(2):
        r = summarize(c, g)
        assert same(arrays(r), ref)
        r.free()
    c.close()


def test_kept_results_of_every_size():
    c = binding.Context(0)
    held = []
    for n in (1, 3000, 90_000, 1_500_000):
        g = graph(n, 2 * n)
        ref = arrays(summarize(c, g))
        held += [(summarize(c, g), ref) for _ in range(6)]
    for r, _ in held[::3]:
        r.free()
    held = [x for i, x in enumerate(held) if i % 3]
    later = [(summarize(c, graph(n, 2 * n)), n) for n in (3000, 90_000)]
    c.close()
    for r, ref in held:
        assert same(arrays(r), ref)
        r.free()
    for r, _ in later:
        r.free()


def test_several_threads_at_once():
    graphs = [graph(n, 2 * n) for n in (1_200_000, 900_001, 5000, 1_200_000)]
    c = binding.Context(0)
    refs = [arrays(summarize(c, g)) for g in graphs]
    c.close()
    wrong = []

    def work(i):
        c = binding.Context(0)
        for _ in range(4):
            r = summarize(c, graphs[i])
            if not same(arrays(r), refs[i]):
                wrong.append(i)
            r.free()
        c.close()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(graphs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong

"""The pinned host memory of results is bounded: callers that keep their results
get ordinary memory once a context, or all the workers of a server together,
have a GiB pinned; kept blocks make room first, and freed ones serve again."""

import ctypes
import threading

import numpy as np
import pytest
import torch

from paper_2111_12493_amd import binding
from paper_2111_12493_amd import graphgen as gg

pytestmark = pytest.mark.gpu
MOST = 1 << 30
N = (1 << 22) + 77          # 48 MiB of hashes and block ids a result


@pytest.fixture(scope="module")
def graph():
    return binding.DeviceGraph(gg.from_edges(N, [0, 5], [1, 6], [0, 0], types=[]))


def summarize(c, g):
    return binding.summarize(c, g, k_max=1, stop_at_fixpoint=False, result_on_host=True)


def pinned(r):
    """Bytes of the result's hashes and block ids that lie in pinned memory."""
    total = 0
    for f, t in (("hashes", ctypes.c_uint64), ("block_ids", ctypes.c_uint32)):
        p = ctypes.cast(getattr(r.ptr.contents, f), ctypes.POINTER(t))
        a = np.ctypeslib.as_array(p, shape=(r.ptr.contents.n_vertices,))
        total += a.nbytes if torch.from_numpy(a.view(np.int8)).is_pinned() else 0
    return total


def check(r, ref):
    for f in ("hashes", "block_ids", "block_sizes"):
        assert np.array_equal(r.fetch(f), ref[f]), f


def test_kept_results(graph):
    c = binding.Context(0)
    first = summarize(c, graph)
    ref = first.to_dict()
    assert pinned(first) == 12 * N
    held = [first] + [summarize(c, graph) for _ in range(25)]
    got = [pinned(r) for r in held]
    assert MOST - 64 * (1 << 20) <= sum(got) <= MOST
    assert got[-1] == 0           # (ordinary memory, as before there was a pool)
    for r in held[::5] + held[-1:]:
        check(r, ref)
    # freed blocks serve later calls
    for r in held[:4]:
        r.free()
    again = [summarize(c, graph) for _ in range(2)]
    assert all(pinned(r) == 12 * N for r in again)
    for r in held[4:] + again:
        r.free()
    # what is kept now makes room for blocks of other sizes
    big = [summarize(c, binding.DeviceGraph(gg.from_edges(10 * N, [0], [1], [0], types=[]))) for _ in range(2)]
    assert sum(pinned(r) for r in big) <= MOST and pinned(big[0]) == 120 * N
    c.close()
    for r in big:
        assert r.fetch("block_ids")[-1] <= 2
        r.free()


def test_results_of_a_server(graph):
    srv = binding.Server(0, workers=3)
    held, lock = [], threading.Lock()

    def submit():
        gs = graph.struct()
        flags = binding.RESULT_ON_HOST
        req = binding.BsimRequest(binding.REQ_SUMMARIZE, 0, ctypes.pointer(gs), binding.BsimParams(1, flags), None, None, 0)
        t = ctypes.c_uint64()
        assert binding.lib().bsim_server_submit(srv.handle, ctypes.byref(req), ctypes.byref(t)) == binding.OK
        r = srv.poll(t.value)[0]
        with lock:
            held.append(r)

    threads = [threading.Thread(target=lambda: [submit() for _ in range(9)]) for _ in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert sum(pinned(r) for r in held) <= MOST
    ref = held[0].to_dict()
    srv.free()
    for r in held:
        check(r, ref)
        r.free()

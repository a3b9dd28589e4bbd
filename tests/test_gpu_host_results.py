"""Results and uploads in host memory: blocks that results give back and later
calls use again (sizes around the pool's steps), results that outlive later
calls and their context, results freed on other threads, small graphs that go
up in one copy and larger ones that do not."""

import threading

import numpy as np
import pytest

from oracle import oracle as orc
from paper_2111_12493_amd import binding
from paper_2111_12493_amd import graphgen as gg

from gpu_util import assert_same

pytestmark = pytest.mark.gpu


def graph(n, m, seed, alive=False):
    rng = np.random.default_rng(seed)
    live = np.ones(n, dtype=np.uint8)
    if alive:
        live[n // 2:: 7] = 0
    ids = np.flatnonzero(live)
    types = [[int(x) for x in rng.integers(0, 5, size=int(c))] if a else [] for c, a in zip(rng.integers(0, 3, n), live)]
    return gg.from_edges(n, rng.choice(ids, m), rng.choice(ids, m), rng.integers(0, 6, m), types=types,
                         alive=live if alive else None)


def run(c, g, host=True):
    return binding.summarize(c, binding.HostGraph(g) if host else binding.DeviceGraph(g), k_max=4,
                             stop_at_fixpoint=False, result_on_host=True)


@pytest.mark.parametrize("u16", [False, True])
@pytest.mark.parametrize("n,m,alive", [(1, 0, False), (2, 1, False), (300, 900, True), (4000, 21001, True),
                                       (60000, 90001, False), (60001, 200003, False)])
def test_uploads_and_results(n, m, alive, u16):
    g = graph(n, m, n + m, alive)
    ref = orc.summarize(g, 4, False)
    c = binding.Context(0)
    for host in (True, False, True):
        r = run(c, gg.with_u16_labels(g) if u16 else g, host)
        assert_same(r.to_dict(), ref, (n, m, host))
        r.free()
    c.close()


def test_blocks_are_not_shared_by_live_results():
    c = binding.Context(0)
    gs = [graph(200 + 37 * i, 700 + 101 * i, i) for i in range(12)]
    refs = [orc.summarize(g, 4, False) for g in gs]
    held = [run(c, g) for g in gs[:6]]
    for r in held[::2]:
        r.free()
    later = [run(c, g) for g in gs[6:]]
    for r, ref in list(zip(held, refs))[1::2] + list(zip(later, refs[6:])):
        assert_same(r.to_dict(), ref)
    threads = [threading.Thread(target=r.free) for r in held[1::2] + later[:3]]
    for t in threads:
        t.start()
    again = [run(c, g) for g in gs[:3]]
    for t in threads:
        t.join()
    for r, ref in zip(again, refs):
        assert_same(r.to_dict(), ref)
    for r in again + later[3:]:
        r.free()
    c.close()


def test_batched_results_share_one_block():
    c = binding.Context(0)
    gs = [graph(50 + 11 * i, 90 + 40 * i, 100 + i) for i in range(20)]
    refs = [orc.summarize(g, g.n + 2, True) for g in gs]
    for _ in range(3):
        rs = binding.batch_summarize(c, [binding.HostGraph(g) for g in gs], result_on_host=True)
        for r in rs[:10]:
            r.free()
        for r, ref in zip(rs[10:], refs[10:]):
            assert_same(r.to_dict(), ref)
    c.close()

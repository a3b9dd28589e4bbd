"""The framework's work as cases to be timed: summaries of small, ordinary and
very large graphs, update batches on a resident summary, many graphs in one
call, and a serving queue.

A case is a dict of plain values.  ``listed()`` names the fixed ones, ``draw``
gives others of the same ranges, ``prepare`` makes what a program holds before
the call, ``run`` is one pass through the public entry points, ``work`` what
the pass cannot do without and ``exact`` the same results in plain torch.

Inputs are drawn on the GPU from the seed: R-MAT graphs (0.57, 0.19, 0.19,
0.05) or uniform ones, edge labels and vertex types by Zipf laws, as in the
repository's own workloads.  Endpoints, labels and types come from tables of
quantized distributions, so that a graph of 2^30 edges takes about a second.
"""

import functools
import math

import numpy as np
import torch

from paper_2111_12493_amd import binding, devgen, graphgen

FIELDS = ("hashes", "block_ids", "block_sizes", "se_src", "se_label", "se_dst")
STATE_FIELDS = FIELDS[:3]   # resident states here keep no summary edges
SIZES = ("k_done", "fixpoint", "n_blocks", "n_summary_edges")
CHUNK = 1 << 26
K_FREE = -1                 # no level cap: to the fixpoint


# ------------------------------------------------------------------ the cases

def _summary(name, kind, n, m, **kw):
    c = {"call": "summarize", "graph": kind, "n": n, "m": m, "u16": False, "labels": 64, "types": 128,
         "chains": 0, "chain_len": 0, "k_max": K_FREE, "stop": True, "untyped": False, "edges": True,
         "direction": "out", "keep_labels": 0, "prev_edges": False, "host": False}
    c.update(kw)
    return dict(c, name=name) if name else c


def _update(name, kind, n, m, k, ops):
    c = {"call": "update", "graph": kind, "n": n, "m": m, "u16": False, "labels": 64, "types": 128,
         "chains": 0, "chain_len": 0, "k_max": k, "ops": ops}
    return dict(c, name=name) if name else c


def _many(name, call, graphs, m_lo, m_hi):
    c = {"call": call, "graphs": graphs, "m_lo": m_lo, "m_hi": m_hi, "labels": 32, "types": 32}
    return dict(c, name=name) if name else c


def listed():
    return [
        # a document-sized graph given as host arrays, results back on the host: latency and launches
        _summary("host_1k", "uniform", 1000, 5003, labels=16, types=8, host=True),
        # the ordinary parity workload, resident on the GPU
        _summary("uniform_10k_50k", "uniform", 10000, 50000, labels=16, types=8),
        # a fresh summary as the serving workload asks for it (degree 8, odd sizes)
        _summary("rmat_1m", "rmat", 125003, 1000003, labels=32, types=32),
        # both edge directions in one signature on a mid-size graph
        _summary("rmat22_both", "rmat", 1 << 22, 1 << 25, direction="both"),
        # long k-chaining: 500 levels, most of which move only the chains
        _summary("rmat20_chains", "rmat", 1 << 20, 1 << 23, types=256, chains=64, chain_len=500),
        # hub-free graph beyond every cache, 16-bit labels
        _summary("uniform24", "uniform", 1 << 24, 1 << 27, u16=True),
        # the SchemEX model (exactly one level) on a large graph
        _summary("rmat24_schemex", "rmat", 1 << 24, 1 << 27, k_max=1, stop=False),
        # the headline workload: 2^30 edges to the fixpoint, capped at 64 levels
        _summary("rmat27", "rmat", 1 << 27, 1 << 30, u16=True, labels=256, types=1024, k_max=64),
        # a small batch of changes on a resident skewed graph, and its undoing
        _update("update_rmat22_2k", "rmat", 1 << 22, 1 << 25, 2, 2000),
        # a large batch on a resident hub-free graph at k = 4, and its undoing
        _update("update_uniform23_100k", "uniform", 1 << 23, 1 << 26, 4, 100000),
        # many small and mid-size graphs in one call
        _many("batch_192", "batch", 192, 100, 300000),
        # a burst of summarize requests to a serving loop of four workers
        _many("serve_16", "serve", 16, 10000, 3000000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["summarize"] * 6 + ["update"] * 2 + ["batch", "serve"])
    if call in ("batch", "serve"):
        top = 300000 if call == "batch" else 3000000
        return _many(None, call, _log_int(rng, 4, 256 if call == "batch" else 24), rng.choice([100, 1000, 10000]),
                     _log_int(rng, 20000, top))
    kind = rng.choice(["rmat", "uniform"])
    if call == "update":
        m = _log_int(rng, 100000, 1 << 26)
        return _update(None, kind, max(64, int(m / rng.uniform(4, 16))), m, rng.randint(1, 4),
                       _log_int(rng, 100, max(200, min(300000, m // 50))))
    m = _log_int(rng, 1000, 1 << 28)
    n = max(16, int(m / rng.uniform(3, 16)))
    c = _summary(None, kind, n, m, u16=rng.random() < 0.5, labels=rng.choice([1, 16, 64, 256]),
                 types=rng.choice([8, 128, 1024]), host=m < 300000 and rng.random() < 0.5)
    form = rng.choice(["fixpoint", "fixpoint", "levels", "model", "direction", "labels", "prev", "chains"])
    if form == "levels":
        c.update(k_max=rng.randint(1, 6), stop=False, edges=rng.random() < 0.5)
    elif form == "model":
        c.update(k_max=rng.choice([0, 1]), stop=False, untyped=rng.random() < 0.5)
    elif form == "direction":
        c.update(direction=rng.choice(["in", "both"]))
    elif form == "labels":
        c.update(keep_labels=max(1, c["labels"] // 2))
    elif form == "prev":
        c.update(k_max=rng.randint(1, 4), stop=False, prev_edges=True)
    elif form == "chains":
        length = _log_int(rng, 16, 400)
        c.update(chains=rng.randint(1, 64), chain_len=length, m=min(m, (1 << 32) // (40 * length)))
        c.update(n=max(16, min(n, c["m"])))
    return c


# ------------------------------------------------------------------ inputs

def _table(p, size, device):
    """size entries, entry i an outcome drawn with probability p (quantized)."""
    cdf = np.cumsum(np.asarray(p, dtype=np.float64))
    at = (np.arange(size) + 0.5) / size * cdf[-1]
    return torch.from_numpy(np.searchsorted(cdf, at).astype(np.int64)).to(device)


@functools.lru_cache(None)
def _zipf_table(k, s):
    return _table(1.0 / np.arange(1, k + 1) ** s, 1 << 20, "cuda").to(torch.int32)


def _zipf(gen, k, s, size):
    tab = _zipf_table(k, s)
    out = torch.empty(size, dtype=torch.int32, device="cuda")
    for lo in range(0, size, CHUNK):
        hi = min(size, lo + CHUNK)
        out[lo:hi] = tab[torch.randint(0, 1 << 20, (hi - lo,), generator=gen, device="cuda", dtype=torch.int32)]
    return out


@functools.lru_cache(None)
def _rmat_table():
    """Three R-MAT levels per entry: the source's three bits << 32 | the target's."""
    p1 = np.array([0.57, 0.19, 0.19, 0.05])
    quad = _table(np.einsum("a,b,c->abc", p1, p1, p1).reshape(-1), 1 << 16, "cuda")
    tab = torch.zeros_like(quad)
    for d in range(3):
        digit = (quad >> (2 * (2 - d))) & 3
        tab = tab * 2 + ((digit >> 1) << 32) + (digit & 1)
    return tab


def _rmat_pairs(gen, n, m):
    """m R-MAT endpoint pairs on the vertices below n as (source, target),
    drawn again where one is n or more."""
    levels = -(-max(1, (n - 1).bit_length()) // 3) * 3
    tab = _rmat_table()
    drop = levels - max(1, (n - 1).bit_length())
    src = torch.empty(m, dtype=torch.int32, device="cuda")
    dst = torch.empty(m, dtype=torch.int32, device="cuda")
    exact = n & (n - 1) == 0
    have = 0
    while have < m:
        c = min(CHUNK, m - have)
        key = torch.zeros(c, dtype=torch.int64, device="cuda")
        for lv in range(0, levels, 9):
            r = torch.randint(0, 1 << 48, (c,), generator=gen, device="cuda", dtype=torch.int64)
            for f in range(min(3, (levels - lv) // 3)):
                key = key * 8 + tab[(r >> (16 * f)) & 0xFFFF]
        s, d = (key >> 32) >> drop, (key & 0xFFFFFFFF) >> drop
        if not exact:
            ok = (s < n) & (d < n)
            s, d = s[ok], d[ok]
        src[have:have + s.numel()] = s
        dst[have:have + s.numel()] = d
        have += s.numel()
    return src, dst


def _graph(case, seed):
    """The case's graph as (source, target, label, type offsets, types), edges by source."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 1000003 + case["m"])
    n, m = case["n"], case["m"]
    if case["graph"] == "rmat":
        src, dst = _rmat_pairs(gen, n, m)
        src, order = torch.sort(src, stable=True)
        dst = dst[order]
        del order
    else:
        src = torch.sort(torch.randint(0, n, (m,), generator=gen, device="cuda", dtype=torch.int32)).values
        dst = torch.randint(0, n, (m,), generator=gen, device="cuda", dtype=torch.int32)
    lab = _zipf(gen, case["labels"], 1.1, m)
    count = torch.randint(0, 5, (n,), generator=gen, device="cuda", dtype=torch.int64)
    typ = None
    if case["chains"]:
        # chains of one further type and label 0, after the other vertices
        per, length = case["chain_len"] + 1, case["chain_len"]
        head = n + per * torch.arange(case["chains"], device="cuda", dtype=torch.int32).repeat_interleave(length)
        step = torch.arange(length, device="cuda", dtype=torch.int32).repeat(case["chains"])
        src, dst = torch.cat([src, head + step]), torch.cat([dst, head + step + 1])
        lab = torch.cat([lab, torch.zeros_like(head)])
        n += per * case["chains"]
        typ = torch.full((per * case["chains"],), case["types"], dtype=torch.int32, device="cuda")
        count = torch.cat([count, torch.ones(per * case["chains"], dtype=torch.int64, device="cuda")])
    toff = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(count, 0, out=toff[1:])
    drawn = _zipf(gen, case["types"], 1.1, int(toff[-1]) - (0 if typ is None else typ.numel()))
    return n, src, dst, lab, toff, drawn if typ is None else torch.cat([drawn, typ])


def _csr(case, g):
    n, src, dst, lab, toff, typ = g
    row = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    for lo in range(0, src.numel(), 4 * CHUNK):
        row[1:] += torch.bincount(src[lo:lo + 4 * CHUNK], minlength=n)
    row = torch.cumsum(row, 0)
    u16 = case.get("u16", False)
    return devgen.DeviceCSR(n=n, m=src.numel(), row_off=row.to(torch.int32), tgt=dst,
                            lab=lab.to(torch.int16) if u16 else lab, type_off=toff.to(torch.int32), typ=typ,
                            label_bytes=2 if u16 else 4, n_labels=case["labels"], n_types=case["types"])


def _on_host(c):
    def host(t, dt):
        return t.cpu().numpy().view(dt)

    return binding.HostGraph(graphgen.Graph(
        n=c.n, row_off=host(c.row_off, np.uint32), tgt=host(c.tgt, np.uint32),
        lab=host(c.lab, np.uint16 if c.label_bytes == 2 else np.uint32), typ_off=host(c.type_off, np.uint32),
        typ=host(c.typ, np.uint32), n_labels=c.n_labels, n_types=c.n_types))


def _parts(case):
    """The graphs of one pass as cases of their own: one, or those of a batch
    or a burst (edges log-uniform, degree 4 to 16; sizes fixed by the case)."""
    if "graphs" not in case:
        return [case]
    rng = np.random.default_rng(case["graphs"])
    out = []
    for _ in range(case["graphs"]):
        m = int(round(math.exp(rng.uniform(math.log(case["m_lo"]), math.log(case["m_hi"])))))
        out.append({"graph": "rmat", "n": max(2, int(round(m / rng.uniform(4, 16)))), "m": m, "chains": 0,
                    "chain_len": 0, "labels": case["labels"], "types": case["types"]})
    return out


def _n_m(part):
    """Vertices and edges of a part, its chains included."""
    return (part["n"] + part["chains"] * (part["chain_len"] + 1), part["m"] + part["chains"] * part["chain_len"])


def _keys(src, dst, lab, n, labels):
    return (src.to(torch.int64) * n + dst) * labels + lab


def _ops(case, g, seed):
    """An update batch as op arrays, and the batch that undoes it.

    60 % edges added, 25 % modified (one in ten a vertex's types, else an
    edge's label), 15 % edges deleted.  Vertices are neither added nor
    deleted: their ids are never used again, so no batch could undo that.
    Added and relabelled triples are new, so the undoing leaves the triples
    that were there.
    """
    n, src, dst, lab, toff, typ = g
    L, m, ops = case["labels"], src.numel(), case["ops"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 31 + 7)
    n_del, n_mod_v = int(ops * 0.15), max(1, int(ops * 0.025))
    n_mod_e = int(ops * 0.25) - n_mod_v
    n_add = ops - n_del - n_mod_v - n_mod_e
    # distinct triples to delete or relabel
    pick = torch.unique(torch.randint(0, m, (2 * (n_del + n_mod_e) + 64,), generator=gen, device="cuda"))
    pick = pick[torch.randperm(pick.numel(), generator=gen, device="cuda")]
    key = _keys(src[pick], dst[pick], lab[pick], n, L)
    first = torch.unique(key, return_inverse=True)[1]
    seen = torch.full((pick.numel(),), pick.numel(), device="cuda").scatter_reduce_(
        0, first, torch.arange(pick.numel(), device="cuda"), "amin")
    pick = pick[seen[first] == torch.arange(pick.numel(), device="cuda")]
    dele, mode = pick[:n_del], pick[n_del:n_del + n_mod_e]
    new_lab = (lab[mode] + torch.randint(1, max(2, L), (mode.numel(),), generator=gen, device="cuda",
                                         dtype=torch.int32)) % L
    if case["graph"] == "rmat":
        a_src, a_dst = _rmat_pairs(gen, n, n_add)
    else:
        a_src = torch.randint(0, n, (n_add,), generator=gen, device="cuda", dtype=torch.int32)
        a_dst = torch.randint(0, n, (n_add,), generator=gen, device="cuda", dtype=torch.int32)
    a_lab = _zipf(gen, L, 1.1, n_add)
    # keep the additions and relabellings whose triple is new, once each
    cand = torch.cat([_keys(a_src, a_dst, a_lab, n, L), _keys(src[mode], dst[mode], new_lab, n, L)])
    new = torch.ones(cand.numel(), dtype=torch.bool, device="cuda")
    order = torch.sort(cand).values
    for lo in range(0, m, CHUNK):
        have = _keys(src[lo:lo + CHUNK], dst[lo:lo + CHUNK], lab[lo:lo + CHUNK], n, L)
        at = torch.searchsorted(order, have).clamp_(max=order.numel() - 1)
        new &= ~torch.isin(cand, have[order[at] == have])
    place = torch.unique(cand, return_inverse=True)[1]
    seen = torch.full((cand.numel(),), cand.numel(), device="cuda").scatter_reduce_(
        0, place, torch.arange(cand.numel(), device="cuda"), "amin")
    new &= seen[place] == torch.arange(cand.numel(), device="cuda")
    add, mod = new[:n_add], new[n_add:]
    a_src, a_dst, a_lab = a_src[add], a_dst[add], a_lab[add]
    mode, new_lab = mode[mod], new_lab[mod]
    verts = torch.unique(torch.randint(0, n, (n_mod_v,), generator=gen, device="cuda"))
    v_cnt = torch.randint(0, 5, (verts.numel(),), generator=gen, device="cuda")
    v_typ = _zipf(gen, case["types"], 1.1, int(v_cnt.sum()))

    def cpu(t):
        return t.cpu().numpy()

    host = {k: cpu(t).astype(np.uint32) for k, t in dict(
        as_=a_src, ad=a_dst, al=a_lab, ms=src[mode], md=dst[mode], ml=lab[mode], mn=new_lab, ds=src[dele],
        dd=dst[dele], dl=lab[dele], v=verts, vc=v_cnt, vt=v_typ).items()}
    old_cnt = cpu(toff[verts + 1] - toff[verts])
    old_at = np.concatenate([np.arange(a, a + c) for a, c in zip(cpu(toff[verts]), old_cnt)] + [np.zeros(0, int)])
    old_typ = cpu(typ[torch.from_numpy(old_at.astype(np.int64)).cuda()]).astype(np.uint32)

    def arrays(added, relabel, deleted, counts, types, rng):
        s, d, l, nl = (np.concatenate(x) for x in (
            (added[0], relabel[0], deleted[0], host["v"]),
            (added[1], relabel[1], deleted[1], 0 * host["v"]),
            (added[2], relabel[2], deleted[2], 0 * host["v"]),
            (0 * added[0], relabel[3], 0 * deleted[0], 0 * host["v"])))
        op = np.concatenate([np.full(x.size, o, dtype=np.uint32) for x, o in (
            (added[0], binding.OP_ADD_E), (relabel[0], binding.OP_MOD_E), (deleted[0], binding.OP_DEL_E),
            (host["v"], binding.OP_MOD_V))])
        cnt = np.concatenate([np.zeros(op.size - counts.size, dtype=np.int64), counts.astype(np.int64)])
        mix = rng.permutation(op.size)   # the kinds of change come mixed
        start = np.cumsum(cnt) - cnt
        ids = np.concatenate([types[start[i]:start[i] + cnt[i]] for i in mix if cnt[i]] + [types[:0]])
        t_off = np.concatenate([[0], np.cumsum(cnt[mix])])
        return dict(op=op[mix], u=s[mix], w=d[mix], label=l[mix], new_label=nl[mix], t_off=t_off, t_ids=ids)

    a = (host["as_"], host["ad"], host["al"])
    r = (host["ms"], host["md"], host["ml"], host["mn"])
    e = (host["ds"], host["dd"], host["dl"])
    rng = np.random.default_rng(seed)
    there = arrays(a, r, e, host["vc"], host["vt"], rng)
    back = arrays(e, (r[0], r[1], r[3], r[2]), a, old_cnt, old_typ, rng)
    after = dict(add=(a_src, a_dst, a_lab), relabel=(mode, new_lab), delete=dele, verts=verts, count=v_cnt, types=v_typ)
    return there, back, after


class Buffers:
    """Arrays that a program keeps for the results, one range per graph: as
    long as the vertices (hashes, block ids, block sizes) and the edges
    (summary edges), of which a result fills the front."""

    def __init__(self, case, fields, on_host):
        sizes = [_n_m(p) for p in _parts(case)]
        self.n = [0] + [int(x) for x in np.cumsum([n for n, _ in sizes])]
        self.m = [0] + [int(x) for x in np.cumsum([m for _, m in sizes])]
        self.kind = binding.MEM_HOST if on_host else binding.MEM_DEVICE
        self.levels = case["k_max"] + 1 if case.get("k_max", K_FREE) >= 0 else case.get("chain_len", 0) + 64
        self.arrays, self.base = {}, {}
        for f in fields:
            count = self.m[-1] if f.startswith("se_") else self.n[-1]
            if on_host:
                self.arrays[f] = np.zeros(count, dtype=binding.Result.FIELDS[f])
                self.base[f] = self.arrays[f].ctypes.data
            else:
                self.arrays[f] = torch.zeros(count, dtype=torch.int64 if f == "hashes" else torch.int32, device="cuda")
                self.base[f] = self.arrays[f].data_ptr()
        self.item = {f: binding.Result.FIELDS[f]().itemsize for f in fields}

    def take(self, results):
        """The results' arrays copied into these, and their sizes."""
        copy = binding.lib().bsim_result_copy
        sizes = np.zeros((len(results), len(SIZES)), dtype=np.int64)
        levels = np.zeros((len(results), self.levels), dtype=np.int64)
        for i, r in enumerate(results):
            for f, base in self.base.items():
                at = (self.m if f.startswith("se_") else self.n)[i]
                rc = copy(r.ptr, f.encode(), base + at * self.item[f], self.kind)
                if rc != binding.OK:
                    raise binding.BsimError(rc, f)
            sizes[i] = [getattr(r, f) for f in SIZES]
            counts = r.blocks_per_iter[:self.levels]
            levels[i, :counts.size] = counts
        return dict(self.arrays, sizes=sizes, blocks_per_iter=levels)


def prepare(case, seed):
    call = case["call"]
    if call == "summarize":
        g = _csr(case, _graph(case, seed))
        torch.cuda.empty_cache()
        return {"case": case, "ctx": binding.Context(0), "graph": _on_host(g) if case["host"] else g,
                "out": Buffers(case, FIELDS if case["edges"] else STATE_FIELDS, case["host"])}
    if call == "update":
        g = _graph(case, seed)
        there, back, _ = _ops(case, g, seed)
        ctx = binding.Context(0)
        c = _csr(case, g)
        state = binding.State(ctx, c, case["k_max"], summary_edges=False)
        del g, c
        torch.cuda.empty_cache()
        return {"case": case, "ctx": ctx, "state": state,
                "batches": [binding.UpdateBatch.from_op_arrays(b) for b in (there, back)],
                "out": [Buffers(case, STATE_FIELDS, False) for _ in range(2)]}
    graphs = [_csr(c, _graph(c, seed * 4099 + i)) for i, c in enumerate(_parts(case))]
    state = {"case": case, "graphs": graphs, "out": Buffers(case, FIELDS, call == "batch")}
    if call == "batch":
        return dict(state, ctx=binding.Context(0))
    return dict(state, server=binding.Server(0, workers=4))


# ------------------------------------------------------------------ one pass

def run(state):
    case = state["case"]
    if case["call"] == "summarize":
        kept = range(case["keep_labels"]) if case["keep_labels"] else None
        r = binding.summarize(state["ctx"], state["graph"],
                              k_max=binding.K_UNBOUNDED if case["k_max"] < 0 else case["k_max"],
                              stop_at_fixpoint=case["stop"], untyped=case["untyped"], summary_edges=case["edges"],
                              result_on_host=case["host"], direction=case["direction"], labels=kept,
                              prev_level_edges=case["prev_edges"])
        return state["out"].take([r])
    if case["call"] == "update":
        # the batch, then the batch that undoes it: the next pass finds the same graph
        return [out.take([state["state"].apply(b)]) for b, out in zip(state["batches"], state["out"])]
    if case["call"] == "batch":
        return state["out"].take(binding.batch_summarize(state["ctx"], state["graphs"], result_on_host=True))
    tickets = [state["server"].submit_summarize(g) for g in state["graphs"]]
    return state["out"].take([state["server"].poll(t)[0] for t in tickets])


def work(case):
    """Every input array read once and every result array written once.  The
    summary edges are counted as one triple per edge (most triples of these
    graphs are distinct); further levels of the refinement are not counted."""
    def graph(n, m, label_bytes, edges=True):
        # two types a vertex; hashes, block ids and block sizes come out
        return 8 * (n + 1) + 4 * 2 * n + m * (4 + label_bytes) + 16 * n + (12 * m if edges else 0)

    if case["call"] == "summarize":
        b = graph(*_n_m(case), 2 if case["u16"] else 4, case["edges"])
    elif case["call"] == "update":
        # two batches read their operations and write hashes, block ids and sizes
        b = 2 * (32 * case["ops"] + 16 * case["n"])
    else:
        b = sum(graph(*_n_m(p), 4) for p in _parts(case))
    return {"bytes": b, "flops": 0}


# ------------------------------------------------------------------ the same in plain torch

def _signed(x):
    return x - (1 << 64) if x >= 1 << 63 else x


def _mix(z):
    """SplitMix64's output function on int64 tensors (wrapping products)."""
    z = (z ^ ((z >> 30) & ((1 << 34) - 1))) * _signed(0xBF58476D1CE4E5B9)
    z = (z ^ ((z >> 27) & ((1 << 37) - 1))) * _signed(0x94D049BB133111EB)
    return z ^ ((z >> 31) & ((1 << 33) - 1))


def _row_sums(f, row, n):
    """Sums of f (ordered by row) per row, modulo 2^64."""
    ends = torch.searchsorted(row, torch.arange(n, device=row.device, dtype=row.dtype), right=True)
    total = torch.cat([torch.zeros(1, dtype=torch.int64, device=f.device), torch.cumsum(f, 0)])
    upto = total[ends]
    return upto - torch.cat([upto.new_zeros(1), upto[:-1]])


def _blocks(h):
    """First-occurrence block ids of equal hashes, and their number."""
    names, inv = torch.unique(h, return_inverse=True)
    first = torch.full((names.numel(),), h.numel(), dtype=torch.int64, device=h.device)
    first.scatter_reduce_(0, inv, torch.arange(h.numel(), device=h.device), "amin")
    rank = torch.empty_like(first)
    rank[torch.argsort(first)] = torch.arange(first.numel(), device=h.device)
    return rank[inv], names.numel()


def _summarize(g, k_max=K_FREE, stop=True, untyped=False, edges=True, direction="out", keep_labels=0,
               prev_edges=False):
    n, src, dst, lab, toff, typ = g
    ct, cl, cs, ce = (_mix(torch.tensor([i], device="cuda")) for i in (1, 2, 3, 4))
    if keep_labels:
        kept = lab < keep_labels
        src, dst, lab = src[kept], dst[kept], lab[kept]
    if untyped:
        t = _mix(ct).expand(n).contiguous()
    else:
        owner = torch.repeat_interleave(torch.arange(n, device="cuda"), toff[1:] - toff[:-1])
        pair = torch.unique((owner << 24) | typ.to(torch.int64))
        t = _mix(ct + _row_sums(_mix(ct ^ (pair & 0xFFFFFF)), pair >> 24, n))
    frm, to, q = src, dst, lab.to(torch.int64)
    if direction == "in":
        frm, to = dst, src
    elif direction == "both":
        frm, to, q = torch.cat([src, dst]), torch.cat([dst, src]), torch.cat([q, q + (1 << 31)])
    salt = _mix(cl + q)
    h = before = t
    counts, k, fixpoint = [torch.unique(h).numel()], 0, False
    while k != k_max and not (stop and fixpoint):
        f = _mix(h[to] ^ salt ^ ce)
        f, order = torch.sort(f)
        row = frm[order]
        row, order = torch.sort(row, stable=True)
        f = f[order]
        again = torch.zeros_like(f, dtype=torch.bool)
        again[1:] = (f[1:] == f[:-1]) & (row[1:] == row[:-1])
        f = f.masked_fill(again, 0)
        before, h = h, _mix(t ^ _mix(cs + _row_sums(f, row, n)))
        k += 1
        counts.append(torch.unique(h).numel())
        fixpoint = counts[-1] == counts[-2]
    ids, nb = _blocks(h)
    out = {"hashes": h, "block_ids": ids.to(torch.int32),
           "block_sizes": torch.bincount(ids, minlength=nb).to(torch.int32)}
    none = torch.zeros(0, dtype=torch.int32, device="cuda")
    se = (none, none, none)
    if edges:
        far, nf = (_blocks(before) if prev_edges else (ids, nb))
        width = int(lab.max()) + 1 if lab.numel() else 1
        tri = torch.unique((ids[src] * width + lab) * nf + far[dst])
        se = tuple(x.to(torch.int32) for x in (tri // nf // width, tri // nf % width, tri % nf))
    out.update(zip(FIELDS[3:], se))
    return out, counts, fixpoint


def _laid_out(case, fields, on_host, results):
    """Results of _summarize in the layout of Buffers.take."""
    out = Buffers(case, fields, on_host)
    sizes = np.zeros((len(results), len(SIZES)), dtype=np.int64)
    levels = np.zeros((len(results), out.levels), dtype=np.int64)
    for i, (r, counts, fixpoint) in enumerate(results):
        for f, a in out.arrays.items():
            at = (out.m if f.startswith("se_") else out.n)[i]
            a[at:at + r[f].numel()] = r[f].cpu().numpy().view(a.dtype) if on_host else r[f]
        sizes[i] = [len(counts) - 1, fixpoint, counts[-1], r["se_src"].numel()]
        levels[i, :len(counts)] = counts[:out.levels]
    return dict(out.arrays, sizes=sizes, blocks_per_iter=levels)


def exact(case, seed):
    call = case["call"]
    if call == "summarize":
        levels = case["chain_len"] + 2 if case["chains"] else 6
        if case["m"] * levels > 6.5e9:
            return None   # too long
        got = _summarize(_graph(case, seed), case["k_max"], case["stop"], case["untyped"], case["edges"],
                         case["direction"], case["keep_labels"], case["prev_edges"])
        return _laid_out(case, FIELDS if case["edges"] else STATE_FIELDS, case["host"], [got])
    if call == "update":
        g = _graph(case, seed)
        n, src, dst, lab, toff, typ = g
        _, _, new = _ops(case, g, seed)
        # delete every copy of the deleted and relabelled triples, then add the new ones
        key = _keys(src, dst, lab, n, case["labels"])
        at, nl = new["relabel"]
        keep = ~torch.isin(key, key[torch.cat([new["delete"], at])])
        a = new["add"]
        edges = [torch.cat(x) for x in ((src[keep], src[at], a[0]), (dst[keep], dst[at], a[1]), (lab[keep], nl, a[2]))]
        owner = torch.repeat_interleave(torch.arange(n, device="cuda"), toff[1:] - toff[:-1])
        left = ~torch.isin(owner, new["verts"])
        owner = torch.cat([owner[left], torch.repeat_interleave(new["verts"], new["count"])])
        owner, order = torch.sort(owner, stable=True)
        typ = torch.cat([typ[left], new["types"]])[order]
        toff = torch.cat([toff.new_zeros(1), torch.cumsum(torch.bincount(owner, minlength=n), 0)])
        there = (n, edges[0], edges[1], edges[2], toff, typ)
        return [_laid_out(case, STATE_FIELDS, False, [_summarize(x, case["k_max"], False, edges=False)])
                for x in (there, g)]
    got = [_summarize(_graph(c, seed * 4099 + i)) for i, c in enumerate(_parts(case))]
    return _laid_out(case, FIELDS, call == "batch", got)

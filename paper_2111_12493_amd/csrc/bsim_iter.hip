// bsim_iter.hip -- the refinement loop (a2-a7).
//
// Level 0 (k_init) hashes every vertex's type set (Algorithm 4's
// initialization: the ID of the local schema) and groups vertices by it.
// Level k >= 1 is then
//   k_iterate  stop test of level k-1 (every block takes the same decision
//              from the level's founded counts; block 0 records it), then
//              h^k: a tile's wave gathers h^{k-1} of its out-edge targets
//              (SignalMessages), de-duplicates the (label, hash) pair keys of
//              each vertex in an LDS table (MergeMessages' hash table), sums
//              the mixed distinct keys (the order-independent Hash) and
//              writes h^k; a hub chunk block writes its mixed keys to the
//              hub's scratch area instead;
//   k_hub      de-duplicates each hub's scratch keys bucket by bucket in LDS,
//              adds each bucket's distinct sum to the hub's accumulator and
//              turns a hub's complete sum into h^k;
//   k_split    the classes of level k: a vertex whose h^k differs from its
//              representative's joins (or founds) the class (rep, h^k) in the
//              split table; the number of founded classes is n_k - n_{k-1}.
//              It also empties the table that level k-1 filled.
// A run that stops at level j hashes no level past it: launch j+1 of
// k_iterate finds the stop.  Past 256 levels of a small graph k_iterate_split
// takes the hashes of level k and the classes of level k-1 in one launch, which
// finds the stop one level later.  The done flag is sticky and later launches
// return at once, so the host can queue launches ahead; block 0 of every
// launch tells the host the class count through a word in host memory.
#include "bsim_device.h"

namespace bsim {

namespace {

// ------------------------------------------------------------ split table

// Join the class (r, key) of the level's split table, founding it if needed.
// A slot holds the owner word ((r + 1) << 32 | owner) of one class; the
// class key is the owner's own key, keys[owner], read back from the level's
// hash array (written by an earlier launch, read-only here).  Returns the
// owner word and sets *founded when this call created the class.  Slots
// only ever go from empty to filled during a launch, so every caller with
// the same (r, key) walks the same probe sequence and stops at the same
// slot; founding a class is one CAS.
__device__ uint64_t split_join(const SplitTable& T, const uint64_t* __restrict__ keys, uint32_t r, uint64_t key,
                               uint32_t v, uint32_t* founded, uint32_t* slot_out) {
    const uint64_t mine = (static_cast<uint64_t>(r + 1) << 32) | v;  // never 0: r + 1 >= 1
    *founded = 0;
    // the home slot depends on the class r as well as the key: isomorphic
    // vertices of different classes (every batched graph has vertices with
    // the same type set) share keys, and must not share one probe chain
    uint32_t slot = (static_cast<uint32_t>(key) ^
                     static_cast<uint32_t>((static_cast<uint64_t>(r) * 0x9E3779B97F4A7C15ull) >> 32)) & T.mask;
    for (;;) {
        uint64_t* p = &T.slots[slot];
        uint64_t cur = *p;  // a stale 0 only costs the CAS below
        if (cur == 0) {
            cur = atomicCAS(reinterpret_cast<unsigned long long*>(p), 0ull, static_cast<unsigned long long>(mine));
            if (cur == 0) {
                *founded = 1;
                *slot_out = slot;
                return mine;
            }
        }
        if ((cur >> 32) == static_cast<uint64_t>(r + 1) && keys[static_cast<uint32_t>(cur)] == key) {
            *slot_out = slot;
            return cur;
        }
        slot = (slot + 1) & T.mask;
    }
}

// split_join for the participating lanes of a wave, with the lanes of one
// (r, key) grouped by ballots first, so that a key shared by many vertices
// (every vertex without out-edges of one type set joins one class) reaches
// the table about once per wave.  The keys of the first kJoinRounds pending
// lanes are grouped; a key held by a large share of the vertices is almost
// surely among them, and the rest go to the table by themselves.  All lanes
// of the wave must call it.  Returns the owner word for participating lanes;
// *founded / *slot as split_join for a group's leader, 0 / 0xFFFFFFFF for
// the others.
__device__ __forceinline__ uint64_t shfl_u64(uint64_t x, uint32_t src) {
    const int lo = __shfl(static_cast<int>(static_cast<uint32_t>(x)), static_cast<int>(src), 64);
    const int hi = __shfl(static_cast<int>(static_cast<uint32_t>(x >> 32)), static_cast<int>(src), 64);
    return (static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32) | static_cast<uint32_t>(lo);
}

constexpr int kJoinRounds = 8;

__device__ uint64_t wave_split_join(const SplitTable& T, const uint64_t* __restrict__ keys, bool participant,
                                    uint32_t r, uint64_t key, uint32_t v, uint32_t* founded, uint32_t* slot_out) {
    const uint32_t lane = lane_id();
    uint32_t leader_of = lane;
    bool pending = participant;
    for (int round = 0; round < kJoinRounds; round++) {
        const uint64_t ball = __ballot(pending);
        if (!ball) break;
        const uint32_t leader = static_cast<uint32_t>(__ffsll(static_cast<long long>(ball)) - 1);
        const uint64_t lk = shfl_u64(key, leader);
        const uint32_t lr = static_cast<uint32_t>(__shfl(static_cast<int>(r), static_cast<int>(leader), 64));
        if (pending && key == lk && r == lr) {
            leader_of = leader;
            pending = false;
        }
    }
    *founded = 0;
    *slot_out = 0xFFFFFFFFu;
    uint64_t o = 0;
    if (participant && leader_of == lane) o = split_join(T, keys, r, key, v, founded, slot_out);
    return shfl_u64(o, leader_of);
}

// base[key] += 1 for every taking lane, one atomic per distinct key in the
// wave (a batched run's founders are counted per graph, and a wave's
// vertices mostly belong to one graph).  All lanes of the wave call it.
__device__ void wave_count_by_key(bool take, uint32_t key, uint32_t* base) {
    const uint32_t lane = lane_id();
    bool pending = take;
    for (;;) {
        const uint64_t ball = __ballot(pending);
        if (!ball) break;
        const uint32_t leader = static_cast<uint32_t>(__ffsll(static_cast<long long>(ball)) - 1);
        const uint32_t lk = static_cast<uint32_t>(__shfl(static_cast<int>(key), static_cast<int>(leader), 64));
        const uint64_t same = __ballot(pending && key == lk);
        if (lane == leader) atomicAdd(&base[lk], static_cast<uint32_t>(__popcll(same)));
        if (key == lk) pending = false;
    }
}

// The claim counter of one stripe at `level`.
__device__ __forceinline__ uint32_t* stripe_of(uint32_t* lcnt, uint32_t level, uint32_t stripe) {
    return lcnt + ((level & (kStripeRing - 1)) * kStripes + stripe) * kStripePitch;
}
__device__ __forceinline__ uint32_t stripe_count(const uint32_t* lcnt, uint32_t level, uint32_t stripe) {
    return lcnt[((level & (kStripeRing - 1)) * kStripes + stripe) * kStripePitch];
}

// Count the classes this wave founded at `level` (up to N per lane, one
// atomic per wave that founded any) and remember their slots so the table
// can be cleared selectively.  All lanes of the wave call it.
template <int N>
__device__ __forceinline__ void record_founders(const SplitTable& T, uint32_t* lcnt, uint32_t level,
                                                const uint32_t (&founded)[N], const uint32_t (&slot)[N]) {
    const uint32_t lane = lane_id();
    uint64_t ball[N];
    uint32_t total = 0;
#pragma unroll
    for (int q = 0; q < N; q++) {
        ball[q] = __ballot(founded[q] != 0);
        total += static_cast<uint32_t>(__popcll(ball[q]));
    }
    if (!total) return;
    const uint32_t stripe = (blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) & (kStripes - 1);
    uint32_t base = 0;
    if (lane == 0) base = atomicAdd(stripe_of(lcnt, level, stripe), total);
    base = static_cast<uint32_t>(__shfl(static_cast<int>(base), 0, 64));
#pragma unroll
    for (int q = 0; q < N; q++) {
        // every counted position is written
        const uint32_t pos = base + static_cast<uint32_t>(__popcll(ball[q] & ((1ull << lane) - 1)));
        if (founded[q] && pos < static_cast<uint32_t>(kListPerStripe))
            T.list[stripe * kListPerStripe + pos] = slot[q];
        base += static_cast<uint32_t>(__popcll(ball[q]));
    }
}

// ------------------------------------------------------------ level 0

// t(v) and h^0 = t for every vertex (0 for a dead one), and the label salts.
__global__ void __launch_bounds__(kBlock) k_types(const uint32_t* __restrict__ type_off,
                                                  const uint32_t* __restrict__ type_ids,
                                                  const uint8_t* __restrict__ alive, uint32_t n, int untyped,
                                                  uint64_t* __restrict__ t, uint64_t* __restrict__ h0,
                                                  uint64_t* __restrict__ salt, uint32_t nsalt, uint32_t in_base) {
    const uint32_t v = blockIdx.x * kBlock + threadIdx.x;
    if (v < nsalt) salt[v] = label_salt(v, in_base);
    if (v < n) {
        uint64_t tv = 0;
        if (!alive || alive[v]) {
            uint64_t sum = 0;
            if (!untyped) {
                const uint32_t a = type_off[v], b = type_off[v + 1];
                for (uint32_t i = a; i < b; i++) {
                    const uint32_t tau = type_ids[i];
                    bool dup = false;
                    for (uint32_t j = a; j < i && !dup; j++) dup = type_ids[j] == tau;
                    if (!dup) sum += mix64(kCT ^ static_cast<uint64_t>(tau));
                }
            }
            tv = mix64(kCT + sum);
        }
        t[v] = tv;
        h0[v] = tv;
    }
}

// Level-0 classes by t (written by k_types, the launch before): many
// vertices share a type set, so each wave's lanes are grouped by key before
// they touch the table.
constexpr int kSplitPerThread = 4;

__global__ void __launch_bounds__(kBlock) k_init(const uint64_t* __restrict__ t, const uint8_t* __restrict__ alive,
                                                 uint32_t n, uint32_t* __restrict__ rep, SplitTable T,
                                                 uint32_t* lcnt, BatchCtl bc) {
    const uint32_t first = blockIdx.x * (kBlock * kSplitPerThread) + threadIdx.x;
    uint32_t founded[kSplitPerThread], slot[kSplitPerThread];
    uint64_t key[kSplitPerThread];
    bool part[kSplitPerThread];
#pragma unroll
    for (int q = 0; q < kSplitPerThread; q++) {
        const uint32_t v = first + q * kBlock;
        part[q] = v < n && (!alive || alive[v]);
        key[q] = part[q] ? t[v] : 0;
    }
#pragma unroll
    for (int q = 0; q < kSplitPerThread; q++) {
        const uint32_t v = first + q * kBlock;
        const uint32_t gi = (part[q] && bc.gid) ? bc.gid[v] : 0u;
        const uint32_t vr = bc.gid ? bc.virt_base + gi : kNoRep;
        const uint64_t o = wave_split_join(T, t, part[q], vr, key[q], v, &founded[q], &slot[q]);
        if (bc.gid) wave_count_by_key(founded[q] != 0, gi, bc.hist);
        if (v < n) rep[v] = part[q] ? static_cast<uint32_t>(o) : 0xFFFFFFFFu;
    }
    record_founders(T, lcnt, 0, founded, slot);
}

// ------------------------------------------------------------ launch k

// Whether level k of graph g of a batched run is this loop's to compute: not
// that of a graph which the small-graph launch has refined to its stop level
// already (its hashes and classes lie in the same arrays), nor one past the
// level at which the graph stopped.  Every block that writes hashes or classes
// of a batched run asks it (k_hub the second half only: see there).
__device__ __forceinline__ bool batch_refines(const BatchCtl& bc, uint32_t g, uint32_t k) {
    return !(bc.ext && bc.ext[g]) && k <= bc.done_level[g];
}

// A wave's keys and table slots, a workgroup's of a solo vertex, or a chunk
// block's bucket counts.
struct WaveLds {
    uint64_t f[kTileMaxEdges];
    uint16_t slot[2 * kTileMaxEdges];
};
struct SoloLds {
    uint64_t f[kSoloMaxEdges];
    uint16_t slot[2 * kSoloMaxEdges];
};
union IterShared {
    WaveLds wave[kWaves];
    SoloLds solo;
    uint32_t hist[(1 << kMaxHubLogB) + 1];
};
static_assert(sizeof(SoloLds) == kWaves * sizeof(WaveLds), "a solo vertex fills the workgroup's LDS exactly");

// Stop test of level k - lag as every wave takes it; true when the run is
// done.  Block 0's first wave also keeps the class count, records the final
// status when the run stops, and reports to the host.
struct StopInputs {
    uint32_t done, cnt, tot;
};
__device__ __forceinline__ StopInputs stop_inputs(const IterArgs& a) {
    StopInputs p{0, 0, 0};
    if (a.hash_only) return p;
    p.done = __hip_atomic_load(&a.status->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (a.k >= a.lag && !a.bc.gid) {
        const uint32_t lv = a.k - a.lag;
        if (lane_id() < static_cast<uint32_t>(kStripes)) p.cnt = stripe_count(a.lcnt, lv, lane_id());
        p.tot = lv ? a.totals[(lv - 1) & (kStripeRing - 1)] : 0u;
    }
    return p;
}
__device__ __forceinline__ bool stop_decision(const IterArgs& a, const StopInputs& p) {
    if (a.hash_only) return false;
    const uint32_t k = a.k;
    uint32_t ex = p.done, fix = 0, nl = 0;
    // batched runs: the per-graph stop launch before this one sets done
    if (!ex && k >= a.lag && !a.bc.gid) {
        const uint32_t lv = k - a.lag;
        const uint32_t c = wave_sum_u32(p.cnt);
        nl = lv == 0 ? c : p.tot + c;
        fix = (lv >= 1 && c == 0) ? 1u : 0u;
        if ((a.stop && fix) || lv >= a.k_max) ex = 1;
        if (threadIdx.x == 0 && blockIdx.x == 0) {
            a.totals[lv & (kStripeRing - 1)] = nl;
            if (ex) {
                a.status->k_done = lv;
                a.status->fixpoint = fix;
                a.status->done = 1;
            }
        }
    }
    if (threadIdx.x == 0 && blockIdx.x == 0 && a.report) {
        const uint32_t flags = (ex ? kReportDone : 0u) | (fix ? kReportFixpoint : 0u) |
                               (a.status->error ? kReportError : 0u);
        // one word: the host needs no ordering between the parts
        __hip_atomic_store(&a.report[k & (kReportRing - 1)],
                           (static_cast<uint64_t>(report_tag(k) | flags) << 32) | nl, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return ex != 0;
}

// kLaneEdges consecutive edges of a lane from edge e on (those at or past m
// are not read): whole vectors where all of them exist, whatever their
// alignment.  Targets and labels are read once per launch: non-temporal, so
// they do not push the gathered hashes out of L2.
template <typename LabT>
__device__ __forceinline__ void load_edges(const uint32_t* __restrict__ tgt, const LabT* __restrict__ lab, uint64_t e,
                                           uint32_t count, uint64_t m, uint32_t (&w)[kLaneEdges],
                                           uint32_t (&l)[kLaneEdges]) {
    typedef uint32_t T4 __attribute__((ext_vector_type(4), aligned(4)));
    typedef uint16_t H8 __attribute__((ext_vector_type(8), aligned(2)));
    if (count && e + kLaneEdges <= m) {
#pragma unroll
        for (int q = 0; q < kLaneEdges; q += 4) {
            const T4 x = __builtin_nontemporal_load(reinterpret_cast<const T4*>(tgt + e + q));
#pragma unroll
            for (int i = 0; i < 4; i++) w[q + i] = x[i];
        }
        if (sizeof(LabT) == 2) {
            const H8 x = __builtin_nontemporal_load(reinterpret_cast<const H8*>(lab + e));
#pragma unroll
            for (int q = 0; q < kLaneEdges; q++) l[q] = x[q];
        } else {
#pragma unroll
            for (int q = 0; q < kLaneEdges; q += 4) {
                const T4 x = __builtin_nontemporal_load(reinterpret_cast<const T4*>(lab + e + q));
#pragma unroll
                for (int i = 0; i < 4; i++) l[q + i] = x[i];
            }
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < kLaneEdges; q++) {
        const bool in = static_cast<uint32_t>(q) < count;
        w[q] = in ? tgt[e + q] : 0u;
        l[q] = in ? static_cast<uint32_t>(lab[e + q]) : 0u;
    }
}

// Table slot of a key in round r (2^kBits slots): a window of the key's bits
// that moves with the round (whole windows of one half, then of the other),
// shifted by the owner, so that equal keys of different vertices of a tile
// never share a slot.
template <int kBits>
__device__ __forceinline__ uint32_t slot_of(uint64_t f, uint32_t owner, uint32_t round) {
    constexpr uint32_t kPer = 32 / kBits;
    const uint32_t half = (round / kPer) & 1 ? static_cast<uint32_t>(f >> 32) : static_cast<uint32_t>(f);
    return ((half >> ((round % kPer) * kBits)) + owner) & ((1u << kBits) - 1);
}

// A tile, by one wave: h^k of up to 64 vertices and 512 edges.
//
// A lane holds eight consecutive edges.  Per edge: gather h^{k-1} of the
// target, mix the pair key, decide whether it is the first of its key in its
// vertex, and sum the first ones per vertex.
//   De-duplication works in rounds on a table of 2-byte slots without
// atomics: every undecided key writes its position to its slot and reads the
// slot back.  The position that stayed is the key's representative if the
// keys are equal (then this one is a repeat), itself if it won, and another
// key otherwise: those keys go to the next round, with another slot.  Equal
// keys of a vertex always share their slots and so never part, and keys of
// earlier rounds no longer matter, so the table is neither cleared nor
// searched.  Every contested slot decides at least one key, so the rounds
// end; at two slots per edge three or four are usual.
//   The sum per vertex is a difference of running sums over the tile's edges
// (mod 2^64), read where a vertex's edges end.
//
// Bound: with hashes in the last-level cache the gather's requests, else its
// DRAM lines.  The workgroup form before (tiles of 1,536 edges, 64-bit
// compare-and-swap per key, a 64-bit LDS add per distinct key, eight
// workgroup barriers, 29 KiB per workgroup of four waves) took 103 us per
// level on R-MAT 2^20 / 2^23 with chains, where this one takes 68; 17.1 and
// 16.3 ms on R-MAT 2^27 / 2^30, 2.64 ms both on 2^24 / 2^27 uniform, where
// nearly every gather is a request past L2 (some 50 G a second of them).
template <typename LabT>
__device__ __forceinline__ void wave_tile(const IterArgs& a, uint32_t tile, WaveLds& L, const StopInputs& p) {
    const uint32_t lane = lane_id();
    const uint4 td = a.tiles[tile];
    // (a queued launch past the stop skips its loads at once)
    const uint32_t nv = p.done ? 0u : td.y - td.x, ne = p.done ? 0u : td.w - td.z;
    const bool mine = lane < nv;
    const uint32_t v = mine ? a.act[td.x + lane] : 0u;
    const uint32_t off = mine ? a.act_off[td.x + lane] - td.z : 0u;
    const uint32_t j0 = lane * kLaneEdges;
    const uint32_t cnt = j0 < ne ? min(ne - j0, static_cast<uint32_t>(kLaneEdges)) : 0u;
    uint32_t w[kLaneEdges], l[kLaneEdges];
    load_edges(a.tgt, static_cast<const LabT*>(a.lab), static_cast<uint64_t>(td.z) + j0, cnt, a.m, w, l);
    uint64_t f[kLaneEdges];
#pragma unroll
    for (int q = 0; q < kLaneEdges; q++) f[q] = static_cast<uint32_t>(q) < cnt ? a.h_prev[w[q]] : 0;
    const uint64_t tv = mine ? a.t[v] : 0;
    bool write = mine;
    if (mine && a.bc.gid) write = batch_refines(a.bc, a.bc.gid[v], a.k);
    const LaneOwners own = lane_owners(reinterpret_cast<uint8_t*>(L.slot), mine, off);
    if (stop_decision(a, p)) return;
    uint32_t todo = 0;
#pragma unroll
    for (int q = 0; q < kLaneEdges; q++) {
        if (static_cast<uint32_t>(q) < cnt) f[q] = mix64(f[q] ^ a.salt[l[q]] ^ kCE);
        // a zero term adds nothing to the sum, repeated or not
        if (static_cast<uint32_t>(q) < cnt && f[q]) todo |= 1u << q;
        L.f[q * 64 + lane] = f[q];
    }
    constexpr int kBits = 10;
    static_assert(2 * kTileMaxEdges == 1 << kBits, "two slots per edge");
    uint32_t first = 0;  // bit q: edge q is the first of its key
    for (uint32_t round = 0; __ballot(todo != 0); round++) {
        wave_sync();
#pragma unroll
        for (int q = 0; q < kLaneEdges; q++)
            if ((todo >> q) & 1) L.slot[slot_of<kBits>(f[q], own.of(q), round)] = static_cast<uint16_t>(q * 64 + lane);
        wave_sync();
        // (a decided key reads what its slot holds too, and drops it)
        uint32_t got[kLaneEdges];
        uint64_t key[kLaneEdges];
#pragma unroll
        for (int q = 0; q < kLaneEdges; q++)
            got[q] = L.slot[slot_of<kBits>(f[q], own.of(q), round)] & (kTileMaxEdges - 1);
#pragma unroll
        for (int q = 0; q < kLaneEdges; q++) key[q] = L.f[got[q]];
        uint32_t won = 0, same = 0;
#pragma unroll
        for (int q = 0; q < kLaneEdges; q++) {
            won |= static_cast<uint32_t>(got[q] == static_cast<uint32_t>(q * 64) + lane) << q;
            same |= static_cast<uint32_t>(key[q] == f[q]) << q;
        }
        first |= todo & won;
        todo &= ~same;  // (the winner reads its own key)
    }
    // running sums of the distinct keys
    uint64_t run = 0;
#pragma unroll
    for (int q = 0; q < kLaneEdges; q++) {
        run += (first >> q) & 1 ? f[q] : 0;
        f[q] = run;
    }
    const uint64_t before = wave_incl_sum(run) - run;
    const bool next_begins = __shfl_down(static_cast<int>(own.starts & 1), 1, 64) != 0;
    wave_sync();
#pragma unroll
    for (int q = 0; q < kLaneEdges; q++) {
        const bool ends = static_cast<uint32_t>(q) < cnt &&
                          (j0 + q + 1 == ne || (q + 1 < kLaneEdges ? own.begins(q + 1) : next_begins));
        if (ends) L.f[own.of(q)] = before + f[q];
    }
    wave_sync();
    // (a tile vertex has edges, so it is alive)
    if (write) {
        const uint64_t sum = L.f[lane] - (lane ? L.f[lane - 1] : 0);
        a.h_next[v] = mix64(tv ^ mix64(kCS + sum));
    }
}

// A hub chunk block: kChunkEdges edges of one hub, their nonzero keys grouped
// by hash bucket (top logb bits) so that each hub-bucket block reads only its
// own keys; the order within a bucket is free.
template <typename LabT>
__device__ void hub_chunk_block(const IterArgs& a, uint32_t blk, IterShared& S, const StopInputs& p) {
    const uint32_t tid = threadIdx.x;
    const uint32_t hi = a.hc_hub[blk];
    const uint32_t e0 = a.hc_e0[blk];
    const uint32_t v = a.hub_v[hi];
    const uint32_t logb = a.hub_logb[hi];
    const uint64_t koff = a.hub_key_off[hi];
    const uint32_t vbeg = a.row_off[v], vend = a.row_off[v + 1];
    const uint32_t ne = p.done ? 0u : min(static_cast<uint32_t>(kChunkEdges), vend - e0);
    const LabT* __restrict__ lab = static_cast<const LabT*>(a.lab);
    uint32_t w[kChunkPerThread];
    uint32_t l[kChunkPerThread];
    uint64_t hv[kChunkPerThread];
#pragma unroll
    for (int r = 0; r < kChunkPerThread; r++) {
        const uint32_t j = tid + r * kBlock;
        w[r] = 0;
        l[r] = 0;
        if (j < ne) {
            w[r] = __builtin_nontemporal_load(&a.tgt[e0 + j]);
            l[r] = static_cast<uint32_t>(__builtin_nontemporal_load(&lab[e0 + j]));
        }
    }
#pragma unroll
    for (int r = 0; r < kChunkPerThread; r++) {
        const uint32_t j = tid + r * kBlock;
        hv[r] = j < ne ? a.h_prev[w[r]] ^ a.salt[l[r]] : 0;
    }
    if (stop_decision(a, p)) return;  // uniform over the block
    uint64_t* __restrict__ out = a.hub_keys + koff + (e0 - vbeg);
    const uint32_t nb = 1u << logb;
    uint32_t* hist = S.hist;
    for (uint32_t b = tid; b <= nb; b += kBlock) hist[b] = 0;
    __syncthreads();
    uint64_t f[kChunkPerThread];
    uint32_t rank[kChunkPerThread];
#pragma unroll
    for (int r = 0; r < kChunkPerThread; r++) {
        const uint32_t j = tid + r * kBlock;
        f[r] = j < ne ? mix64(hv[r] ^ kCE) : 0;
        rank[r] = 0;
        if (f[r] != 0) {
            const uint32_t b = logb ? static_cast<uint32_t>(f[r] >> (64 - logb)) : 0u;
            rank[r] = atomicAdd(&hist[b], 1u);
        }
    }
    __syncthreads();
    if (tid < 64) {  // exclusive prefix over at most 256 buckets, by one wave
        uint32_t run = 0;
        for (uint32_t b0 = 0; b0 < nb; b0 += 64) {
            const uint32_t c = b0 + tid < nb ? hist[b0 + tid] : 0u;
            const uint32_t incl = wave_incl_sum(c);
            if (b0 + tid < nb) hist[b0 + tid] = run + incl - c;
            run += static_cast<uint32_t>(__shfl(static_cast<int>(incl), 63, 64));
        }
        if (tid == 0) hist[nb] = run;
    }
    __syncthreads();
    uint32_t* boff = a.hub_boff + static_cast<uint64_t>(blk) * kHubOffStride;
    for (uint32_t b = tid; b <= nb; b += kBlock) boff[b] = hist[b];
#pragma unroll
    for (int r = 0; r < kChunkPerThread; r++) {
        if (f[r] != 0) {
            const uint32_t b = logb ? static_cast<uint32_t>(f[r] >> (64 - logb)) : 0u;
            out[hist[b] + rank[r]] = f[r];
        }
    }
}

// A vertex of more edges than a tile holds and at most kSoloMaxEdges: the
// rounds of wave_tile over the workgroup, all keys of one owner.
template <typename LabT>
__device__ void solo_block(const IterArgs& a, uint32_t v, SoloLds& L, const StopInputs& p) {
    __shared__ uint64_t s_sum[kWaves];
    const uint32_t tid = threadIdx.x;
    const uint32_t e0 = a.row_off[v];
    const uint32_t ne = p.done ? 0u : a.row_off[v + 1] - e0;
    bool write = tid == 0;
    if (a.bc.gid) write = write && batch_refines(a.bc, a.bc.gid[v], a.k);
    const uint64_t tv = a.t[v];
    const LabT* __restrict__ lab = static_cast<const LabT*>(a.lab);
    uint32_t w[kLaneEdges];
    uint32_t l[kLaneEdges];
    uint64_t f[kLaneEdges];
#pragma unroll
    for (int r = 0; r < kLaneEdges; r++) {
        const uint32_t j = tid + r * kBlock;
        w[r] = 0;
        l[r] = 0;
        if (j < ne) {
            w[r] = __builtin_nontemporal_load(&a.tgt[e0 + j]);
            l[r] = static_cast<uint32_t>(__builtin_nontemporal_load(&lab[e0 + j]));
        }
    }
#pragma unroll
    for (int r = 0; r < kLaneEdges; r++) f[r] = tid + r * kBlock < ne ? a.h_prev[w[r]] ^ a.salt[l[r]] : 0;
    if (stop_decision(a, p)) return;  // uniform over the block
    constexpr int kBits = 12;
    static_assert(2 * kSoloMaxEdges == 1 << kBits, "two slots per edge");
    uint32_t todo = 0;
#pragma unroll
    for (int r = 0; r < kLaneEdges; r++) {
        const uint32_t j = tid + r * kBlock;
        if (j < ne) {
            f[r] = mix64(f[r] ^ kCE);
            L.f[j] = f[r];
            if (f[r]) todo |= 1u << r;
        }
    }
    uint64_t acc = 0;
    for (uint32_t round = 0; __syncthreads_or(todo != 0); round++) {
#pragma unroll
        for (int r = 0; r < kLaneEdges; r++)
            if ((todo >> r) & 1) L.slot[slot_of<kBits>(f[r], 0, round)] = static_cast<uint16_t>(tid + r * kBlock);
        __syncthreads();
        uint32_t got[kLaneEdges];
        uint64_t key[kLaneEdges];
#pragma unroll
        for (int r = 0; r < kLaneEdges; r++) got[r] = L.slot[slot_of<kBits>(f[r], 0, round)] & (kSoloMaxEdges - 1);
#pragma unroll
        for (int r = 0; r < kLaneEdges; r++) key[r] = L.f[got[r]];
#pragma unroll
        for (int r = 0; r < kLaneEdges; r++) {
            if (!((todo >> r) & 1)) continue;
            if (got[r] == tid + r * kBlock) acc += f[r];
            if (key[r] == f[r]) todo &= ~(1u << r);
        }
    }
    acc = wave_sum_u64(acc);
    if (lane_id() == 0) s_sum[tid >> 6] = acc;
    __syncthreads();
    if (write) {
        uint64_t sum = 0;
        for (int i = 0; i < kWaves; i++) sum += s_sum[i];
        a.h_next[v] = mix64(tv ^ mix64(kCS + sum));
    }
}

// kIsoPerBlock vertices without out-edges: h^k = M(t ^ M(C_S)) for every
// k >= 1, written where the hash buffer does not hold it yet.
__device__ void iso_block(const IterArgs& a, uint32_t blk, const StopInputs& p) {
    const uint32_t tid = threadIdx.x;
    if (stop_decision(a, p)) return;
    uint32_t v[kIsoPerThread];
    uint64_t tv[kIsoPerThread];
    bool mine[kIsoPerThread], live[kIsoPerThread];
#pragma unroll
    for (int r = 0; r < kIsoPerThread; r++) {
        const uint32_t i = blk * kIsoPerBlock + r * kBlock + tid;
        mine[r] = i < a.n_iso;
        v[r] = mine[r] ? a.iso[i] : 0u;
        tv[r] = 0;
        live[r] = false;
        if (mine[r]) {
            live[r] = !a.alive || a.alive[v[r]];
            if (a.bc.gid) mine[r] = batch_refines(a.bc, a.bc.gid[v[r]], a.k);
            tv[r] = a.t[v[r]];
        }
    }
#pragma unroll
    for (int r = 0; r < kIsoPerThread; r++)
        if (mine[r]) a.h_next[v[r]] = live[r] ? mix64(tv[r] ^ mix64(kCS)) : 0;
}

// Workgroup b of the hashes of level k.
template <typename LabT>
__device__ __forceinline__ void hash_block(const IterArgs& a, IterShared& S, const StopInputs& p, uint32_t b) {
    if (b < a.n_hub_chunks) {
        hub_chunk_block<LabT>(a, b, S, p);
        return;
    }
    b -= a.n_hub_chunks;
    if (b < a.n_solo) {
        solo_block<LabT>(a, a.solo_v[b], S.solo, p);
        return;
    }
    b -= a.n_solo;
    if (b < a.n_iso_blocks) {
        iso_block(a, b, p);
        return;
    }
    b -= a.n_iso_blocks;
    // one tile per wave (the tile number is the same in all its lanes)
    const uint32_t wv = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)));
    const uint32_t tile = b * kWaves + wv;
    if (tile < a.n_tiles)
        wave_tile<LabT>(a, tile, S.wave[wv], p);
    else
        (void)stop_decision(a, p);  // (an empty graph still needs its stop test)
}

template <typename LabT>
__global__ void __launch_bounds__(kBlock) k_iterate(IterArgs a) {
    __shared__ IterShared S;
    const StopInputs p = stop_inputs(a);  // loaded together with everything else
    const uint32_t b = blockIdx.x;
    if (a.stop_only) {
        (void)stop_decision(a, p);
        return;
    }
    hash_block<LabT>(a, S, p, b);
}

// ------------------------------------------------------------ classes of level k

// Empty the table that level k-1 filled, from the list of its claimed slots
// (one stripe after the other per block), or whole when a list overflowed;
// and the counters that level k+1 will use.
__device__ void recycle(const SplitArgs& a, uint32_t block, uint32_t blocks) {
    const uint32_t tid = threadIdx.x, k = a.k;
    if (block == 0 && tid < kStripes) *stripe_of(a.lcnt, k + 1, tid) = 0;
    const uint32_t mine = stripe_count(a.lcnt, k - 1, tid & (kStripes - 1));
    if (__ballot(mine > static_cast<uint32_t>(kListPerStripe))) {
        const uint64_t cap = static_cast<uint64_t>(a.clr_tab.mask) + 1;
        const uint64_t per = (cap + blocks - 1) / blocks;
        const uint64_t lo = per * block, hi = min(cap, lo + per);
        for (uint64_t j = lo + tid; j < hi; j += kBlock) a.clr_tab.slots[j] = 0;
        return;
    }
    for (uint32_t st = block; st < static_cast<uint32_t>(kStripes); st += blocks) {
        const uint32_t c = stripe_count(a.lcnt, k - 1, st);
        for (uint32_t e = tid; e < c; e += kBlock) {
            const uint32_t idx = a.clr_tab.list[st * kListPerStripe + e];
            if (idx <= a.clr_tab.mask) a.clr_tab.slots[idx] = 0;
        }
    }
}

// Split test of level k.  At level 1 every vertex takes it; from level 2 on
// a vertex without out-edges cannot leave its class (its hash is the same
// function of t at every level >= 1), so the tile vertices and the hubs do.
// A vertex that is its class's representative, as nearly all are once a
// graph has mostly classes of one, costs the 4 bytes of rep alone.
//
// Bound: rep streamed, h of the non-representatives gathered, and at level 1
// the claims (a random 8-byte line each).  It runs as a launch of its own
// because the next launch then knows the level's class count before it
// hashes: with the test inside the next level's hashing launch, every run
// hashed one level that the fixpoint test discarded, and each tile block
// carried the test's four dependent loads and its barriers.  On 2^24 vertices
// and 2^27 edges of a uniform graph a level of both took 3.1 ms and the
// discarded level as much; hashing alone takes 2.65 ms, the split 0.93 ms at
// level 1 and 0.04-0.08 ms from there on.
__device__ __forceinline__ void split_block(const SplitArgs& a, uint32_t block, uint32_t blocks) {
    const uint32_t first = block * (kBlock * kSplitPerThread) + threadIdx.x;
    const uint32_t k = a.k;
    uint32_t v[kSplitPerThread], r[kSplitPerThread], gi[kSplitPerThread];
    uint64_t hv[kSplitPerThread], hr[kSplitPerThread];
    bool probe[kSplitPerThread];
#pragma unroll
    for (int q = 0; q < kSplitPerThread; q++) {
        const uint32_t i = first + q * kBlock;
        probe[q] = i < a.count;
        v[q] = 0;
        if (!probe[q]) continue;
        if (k == 1)
            v[q] = i;
        else if (i < a.n_act)
            v[q] = a.act[i];
        else
            v[q] = i - a.n_act < a.n_solo ? a.solo_v[i - a.n_act] : a.hub_v[i - a.n_act - a.n_solo];
    }
#pragma unroll
    for (int q = 0; q < kSplitPerThread; q++) {
        r[q] = probe[q] ? a.rep[v[q]] : 0u;
        gi[q] = 0;
        if (probe[q] && a.bc.gid) {
            gi[q] = a.bc.gid[v[q]];
            probe[q] = batch_refines(a.bc, gi[q], k);
        }
        probe[q] = probe[q] && r[q] != v[q] && r[q] != 0xFFFFFFFFu;  // (a dead vertex has no class)
    }
#pragma unroll
    for (int q = 0; q < kSplitPerThread; q++) {
        hv[q] = hr[q] = 0;
        if (probe[q]) {
            hv[q] = a.h[v[q]];
            hr[q] = a.h[r[q]];
        }
    }
    uint32_t founded[kSplitPerThread], slot[kSplitPerThread];
#pragma unroll
    for (int q = 0; q < kSplitPerThread; q++) {
        const bool part = probe[q] && hv[q] != hr[q];
        founded[q] = 0;
        slot[q] = 0xFFFFFFFFu;
        uint64_t o = 0;
        if (k == 1)
            o = wave_split_join(a.test_tab, a.h, part, r[q], hv[q], v[q], &founded[q], &slot[q]);
        else if (part)
            o = split_join(a.test_tab, a.h, r[q], hv[q], v[q], &founded[q], &slot[q]);
        if (part) a.rep[v[q]] = static_cast<uint32_t>(o);
        if (a.bc.gid) wave_count_by_key(founded[q] != 0, gi[q], a.bc.hist + static_cast<size_t>(k) * a.bc.n_graphs);
    }
    record_founders(a.test_tab, a.lcnt, k, founded, slot);
    recycle(a, block, blocks);
}

__global__ void __launch_bounds__(kBlock) k_split(SplitArgs a) {
    if (a.status->done) return;
    split_block(a, blockIdx.x, gridDim.x);
}

// Launch k of a deep run: the hashes of level k by the first n_hash workgroups
// (none past k_max) and the class test of level k-1 by the others, which read
// the same level and write nothing that the first ones read.  The stop test is
// that of level k-2.  A level of 20,000 vertices then takes 7.5 us instead of 7.8
// and 4.6 in two launches.
template <typename LabT>
__global__ void __launch_bounds__(kBlock) k_iterate_split(IterArgs a, SplitArgs sp, uint32_t n_hash) {
    __shared__ IterShared S;
    const StopInputs p = stop_inputs(a);
    if (blockIdx.x < n_hash)
        hash_block<LabT>(a, S, p, blockIdx.x);
    else if (!stop_decision(a, p))
        split_block(sp, blockIdx.x - n_hash, gridDim.x - n_hash);
}

// ------------------------------------------------------------ hub buckets

// One workgroup per hash bucket of a hub: the bucket's keys, one run per chunk
// of the hub, are de-duplicated and their sum added to the hub's; the
// workgroup that finishes a hub's last bucket turns the sum into h^k.
//
// A bucket of at most hub_rounds_cap keys, as the schedule aims at, goes
// through the rounds of wave_tile (keys and 2-byte slots in LDS, no atomics).
// Larger ones (a hub past 2^8 buckets, a key repeated very often) go to a
// 64-bit open-addressing table whose distinct keys are counted, and are
// re-split by further hash bits when the count passes the table's limit.
//
// Bound at few hubs: a chain of dependent loads (schedule, run bounds, keys)
// and the rounds' barriers.  With the table alone, whose distinct count is
// one LDS counter, a serial prefix over the runs and a second launch to
// finish the hubs, a level took 29.5 + 4.8 us on R-MAT 2^20 / 2^23; now 12.6.
// On 2^27 / 2^30, with thousands of buckets in flight, 2.48 and 2.30 ms.
constexpr uint32_t kMaxHubRuns = kHubBlock;  // chunk runs staged in LDS at a time

struct HubRuns {
    uint32_t at[kMaxHubRuns + 1];  // exclusive prefix of the run lengths
    uint32_t src[kMaxHubRuns];     // scratch offset of each run
    uint32_t red[kHubBlock / 64];
};

// Stage the runs of chunks [cb, cb + ncb) of this bucket; returns their keys.
__device__ uint32_t stage_runs(const HubArgs& a, uint32_t c0, uint32_t cb, uint32_t ncb, uint32_t bucket,
                               uint32_t e_first, HubRuns& R) {
    const uint32_t tid = threadIdx.x;
    uint32_t len = 0;
    __syncthreads();
    if (tid < ncb) {
        const uint32_t blk = c0 + cb + tid;
        const uint32_t* boff = a.hub_boff + static_cast<uint64_t>(blk) * kHubOffStride;
        const uint32_t b0 = boff[bucket];
        R.src[tid] = (a.hc_e0[blk] - e_first) + b0;
        len = boff[bucket + 1] - b0;
    }
    const uint32_t incl = wave_incl_sum(len);
    if (lane_id() == 63) R.red[tid >> 6] = incl;
    __syncthreads();
    uint32_t base = 0, total = 0;
    for (uint32_t i = 0; i < kHubBlock / 64; i++) {
        if (i < (tid >> 6)) base += R.red[i];
        total += R.red[i];
    }
    if (tid < ncb) R.at[tid] = base + incl - len;
    if (tid == 0) R.at[ncb] = total;
    __syncthreads();
    return total;
}

// Key j of the staged runs.
__device__ __forceinline__ uint64_t run_key(const HubRuns& R, uint32_t ncb, const uint64_t* __restrict__ keys,
                                            uint32_t j) {
    uint32_t lo = 0, hi = ncb;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (R.at[mid] <= j) lo = mid; else hi = mid;
    }
    return keys[R.src[lo] + (j - R.at[lo])];
}

// Sum of the distinct keys of a staged bucket that fits: this thread's share.
__device__ uint64_t hub_rounds(const HubArgs& a, const HubRuns& R, uint32_t ncb, uint32_t total,
                               const uint64_t* __restrict__ keys, uint64_t* s_mem) {
    const uint32_t tid = threadIdx.x;
    const uint32_t cap = hub_rounds_cap(a.table_slots), mask = a.table_slots - 1;
    const uint32_t bits = static_cast<uint32_t>(__popc(mask)), per = 32 / bits;
    uint64_t* lf = s_mem;
    uint16_t* slot = reinterpret_cast<uint16_t*>(s_mem + cap);
    static_assert(kHubRoundsMax <= 32, "a bit per key of a thread");
    uint32_t todo = 0;
    for (uint32_t r = 0, j = tid; j < total; r++, j += kHubBlock) {
        lf[j] = run_key(R, ncb, keys, j);  // (a zero key is not in the scratch)
        todo |= 1u << r;
    }
    uint64_t acc = 0;
    for (uint32_t round = 0; __syncthreads_or(todo != 0); round++) {
        const uint32_t sh = (round % per) * bits;
        const bool upper = (round / per) & 1;
        auto at = [&](uint64_t f) {
            return ((upper ? static_cast<uint32_t>(f >> 32) : static_cast<uint32_t>(f)) >> sh) & mask;
        };
        for (uint32_t left = todo; left; left &= left - 1) {
            const uint32_t j = (static_cast<uint32_t>(__ffs(static_cast<int>(left))) - 1) * kHubBlock + tid;
            slot[at(lf[j])] = static_cast<uint16_t>(j);
        }
        __syncthreads();
        for (uint32_t left = todo; left; left &= left - 1) {
            const uint32_t bit = left & (0u - left);
            const uint32_t j = (static_cast<uint32_t>(__ffs(static_cast<int>(left))) - 1) * kHubBlock + tid;
            const uint64_t f = lf[j];
            const uint32_t got = slot[at(f)];
            if (got == j) acc += f;
            if (lf[got] == f) todo &= ~bit;
        }
    }
    return acc;
}

// The same for a bucket of any size: see k_hub.
__device__ uint64_t hub_table(const HubArgs& a, HubRuns& R, uint32_t c0, uint32_t nc, uint32_t bucket, uint32_t logb,
                              uint32_t e_first, const uint64_t* __restrict__ keys, uint64_t* s_tab) {
    __shared__ uint32_t s_ctl[2];
    const uint32_t tid = threadIdx.x;
    const uint32_t mask = a.table_slots - 1;
    volatile uint32_t* ctl = s_ctl;
    // Only distinct keys occupy slots; a bucket with more distinct keys than
    // the table limit is re-split by further hash bits and re-read, which
    // ends because distinct keys differ in some bit (depth capped for safety).
    uint64_t sum = 0;
    for (uint32_t extra = 0;; extra++) {
        if (extra > kMaxHubExtraBits) {
            if (tid == 0) atomicOr(&a.status->error, kErrHubSplit);
            break;
        }
        sum = 0;
        bool overflow = false;
        const uint32_t bits = logb + extra;
        for (uint32_t sub = 0; sub < (1u << extra) && !overflow; sub++) {
            const uint64_t want = (static_cast<uint64_t>(bucket) << extra) | sub;
            __syncthreads();
            for (uint32_t j = tid; j < a.table_slots; j += kHubBlock) s_tab[j] = 0;
            if (tid == 0) {
                ctl[0] = 0;  // distinct keys inserted
                ctl[1] = 0;  // overflow
            }
            for (uint32_t cb = 0; cb < nc && !overflow; cb += kMaxHubRuns) {
                const uint32_t ncb = min(kMaxHubRuns, nc - cb);
                const uint32_t total = stage_runs(a, c0, cb, ncb, bucket, e_first, R);
                for (uint32_t j0 = 0; j0 < total; j0 += 4 * kHubBlock) {
                    if (ctl[1]) break;
                    uint64_t f[4];
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const uint32_t j = j0 + r * kHubBlock + tid;
                        f[r] = j < total ? run_key(R, ncb, keys, j) : 0;
                    }
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        if (f[r] == 0) continue;
                        if (extra && (f[r] >> (64 - bits)) != want) continue;
                        const uint32_t got =
                            lds_insert_bounded(s_tab, static_cast<uint32_t>(f[r]) & mask, a.table_slots, f[r]);
                        if (got == 1u) {
                            sum += f[r];
                            // count distinct keys only: duplicates never overflow
                            if (atomicAdd(const_cast<uint32_t*>(&ctl[0]), 1u) + 1 >= a.table_limit) ctl[1] = 1;
                        } else if (got == 2u) {
                            ctl[1] = 1;
                        }
                    }
                }
                __syncthreads();
                overflow = ctl[1] != 0;
            }
        }
        if (!overflow) break;
    }
    return sum;
}

__global__ void __launch_bounds__(kHubBlock) k_hub(HubArgs a) {
    extern __shared__ uint64_t s_mem[];
    __shared__ uint64_t s_red64[kHubBlock / 64];
    __shared__ HubRuns R;
    const uint32_t tid = threadIdx.x;
    if (*reinterpret_cast<volatile uint32_t*>(&a.status->done)) return;
    const uint32_t hi = a.hb_hub[blockIdx.x];
    const uint32_t bucket = a.hb_bucket[blockIdx.x];
    const uint32_t logb = a.hub_logb[hi];
    const uint32_t c0 = a.hub_chunk0[hi], nc = a.hub_nchunks[hi];
    const uint64_t* __restrict__ keys = a.hub_keys + a.hub_key_off[hi];
    const uint32_t e_first = a.hc_e0[c0];
    uint64_t sum;
    const uint32_t total = nc <= kMaxHubRuns ? stage_runs(a, c0, 0, nc, bucket, e_first, R) : 0xFFFFFFFFu;
    if (total <= hub_rounds_cap(a.table_slots))
        sum = hub_rounds(a, R, nc, total, keys, s_mem);
    else
        sum = hub_table(a, R, c0, nc, bucket, logb, e_first, keys, s_mem);
    sum = wave_sum_u64(sum);
    if (lane_id() == 0) s_red64[tid >> 6] = sum;
    __syncthreads();
    if (tid != 0) return;
    uint64_t bsum = 0;
    for (int i = 0; i < kHubBlock / 64; i++) bsum += s_red64[i];
    // The hub's sum, then its count of finished buckets.  Both are device
    // atomics and the second is issued once the first has returned, so the
    // workgroup that counts the last bucket reads the whole sum, without
    // fences (an agent-scope fence on this chip writes back or invalidates
    // the whole L2 of the block's XCD).  It clears both for the next level.
    unsigned long long* acc = reinterpret_cast<unsigned long long*>(a.hub_acc) + 2ull * hi;
    const uint64_t was = __hip_atomic_fetch_add(acc, static_cast<unsigned long long>(bsum), __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::"v"(was) : "memory");
    const uint64_t n_done = __hip_atomic_fetch_add(acc + 1, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (n_done + 1 != (1ull << logb)) return;
    asm volatile("s_waitcnt vmcnt(0)" ::"v"(n_done) : "memory");
    const uint64_t all = __hip_atomic_fetch_add(acc, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    acc[0] = 0;
    acc[1] = 0;
    const uint32_t v = a.hub_v[hi];
    // (batch_refines: no graph of the small-graph launch has a hub)
    static_assert(kSmallMaxEdges <= kSoloMaxEdges, "a graph that fits the small-graph launch has no hub");
    if (!a.bc.gid || a.k <= a.bc.done_level[a.bc.gid[v]]) a.h_next[v] = mix64(a.t[v] ^ mix64(kCS + all));
}

// ------------------------------------------------------------ batched stop

// Launch k of a batched run begins with this: graph g stops at level k-lag
// when its class count did not grow there (fixpoint) or k-lag reaches k_max.
__global__ void __launch_bounds__(kBlock) k_graph_stop(BatchCtl bc, uint32_t k, uint32_t lag, uint32_t k_max,
                                                       uint32_t stop, RunStatus* status) {
    const uint32_t g = blockIdx.x * kBlock + threadIdx.x;
    if (g >= bc.n_graphs || k < lag || bc.done_level[g] != 0xFFFFFFFFu) return;
    const uint32_t lv = k - lag;
    const uint32_t c = bc.hist[static_cast<size_t>(lv) * bc.n_graphs + g];
    const uint32_t fx = (lv >= 1 && c == 0) ? 1u : 0u;
    if ((stop && fx) || lv >= k_max) {
        bc.done_level[g] = lv;
        bc.fix[g] = fx;
        if (atomicAdd(bc.n_done, 1u) + 1 == bc.n_graphs) {
            status->k_done = lv;
            status->fixpoint = fx;
            status->done = 1;
        }
    }
}

}  // namespace

uint32_t query_hub_table_slots(int device, bool device_max) {
    int bytes = 0;
    if (hipDeviceGetAttribute(&bytes, hipDeviceAttributeMaxSharedMemoryPerBlock, device) != hipSuccess)
        bytes = 65536;
    // keep room for the block's static LDS.  Keys arrive grouped by bucket,
    // so small tables cost no extra reads and let several blocks share a CU.
    uint64_t avail = bytes > 4096 ? static_cast<uint64_t>(bytes) - 4096 : 4096;
    uint64_t slots = std::min<uint64_t>(avail / 8, device_max ? kHubTableMax : kHubTableDefault);
    uint32_t p = 1;
    while (2ull * p <= slots) p <<= 1;
    return p;
}

static SplitTable make_table(Arena& arena, uint64_t cap) {
    SplitTable T;
    T.slots = arena.alloc<uint64_t>(cap);
    T.list = arena.alloc<uint32_t>(static_cast<size_t>(kStripes) * kListPerStripe);
    T.mask = static_cast<uint32_t>(cap - 1);
    return T;
}

// Clear up to kClearRanges ranges in one launch (a level-0 setup clears six,
// and a launch apiece costs more than the small ones' bytes).
constexpr int kClearRanges = 8;
struct ClearArgs {
    uint4* p[kClearRanges];
    uint64_t n[kClearRanges];  // 16-byte words (allocations are 256-byte multiples)
};

__global__ void __launch_bounds__(kBlock) k_clear(ClearArgs a) {
    const uint64_t first = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const uint64_t step = static_cast<uint64_t>(gridDim.x) * kBlock;
#pragma unroll
    for (int i = 0; i < kClearRanges; i++)
        for (uint64_t j = first; j < a.n[i]; j += step) a.p[i][j] = make_uint4(0, 0, 0, 0);
}

void alloc_run_buffers(const Staged& g, RunBuffers& rb, Arena& arena, hipStream_t s) {
    const uint32_t n = g.n;
    rb.t = arena.alloc<uint64_t>(n);
    rb.h[0] = arena.alloc<uint64_t>(n);
    rb.h[1] = arena.alloc<uint64_t>(n);
    rb.rep = arena.alloc<uint32_t>(n);
    const uint64_t cap = split_table_slots(n);
    ClearArgs c{};
    int nc = 0;
    uint64_t words = 0;
    auto clear = [&](void* p, uint64_t bytes) {
        c.p[nc] = static_cast<uint4*>(p);
        c.n[nc] = (bytes + 15) / 16;
        words = std::max(words, c.n[nc++]);
    };
    for (int i = 0; i < 2; i++) {
        rb.tab[i] = make_table(arena, cap);
        clear(rb.tab[i].slots, cap * sizeof(uint64_t));
    }
    rb.lcnt = arena.alloc<uint32_t>(kStripeRing * kStripes * kStripePitch);
    rb.totals = arena.alloc<uint32_t>(kStripeRing);
    rb.hub_keys = arena.alloc<uint64_t>(g.hub_keys_total + 1);
    rb.hub_boff = arena.alloc<uint32_t>((static_cast<size_t>(g.n_hub_chunks) + 1) * kHubOffStride);
    rb.hub_acc = arena.alloc<uint64_t>(2ull * g.n_hubs + 2);
    rb.status = arena.alloc<RunStatus>(1);
    clear(rb.lcnt, kStripeRing * kStripes * kStripePitch * 4);
    clear(rb.hub_acc, (g.n_hubs + 1) * 16ull);
    clear(rb.status, sizeof(RunStatus));
    k_clear<<<std::min<uint32_t>(ceil_div(words, kBlock), 8192), kBlock, 0, s>>>(c);
    hip_check(hipGetLastError(), "clear run buffers");
}

void launch_init(const Staged& g, const RunBuffers& rb, bool untyped, hipStream_t s) {
    const uint32_t n = g.n;
    const uint32_t nsalt = g.max_label + 1;
    k_types<<<ceil_div(std::max(n, nsalt), kBlock), kBlock, 0, s>>>(g.type_off, g.type_ids, g.alive, n,
                                                                    untyped ? 1 : 0, rb.t, rb.h[0], g.salt, nsalt,
                                                                    g.in_label_base);
    k_init<<<std::max<uint32_t>(ceil_div(n, kBlock * kSplitPerThread), 1), kBlock, 0, s>>>(rb.t, g.alive, n, rb.rep, rb.tab[0], rb.lcnt, rb.bc);
    hip_check(hipGetLastError(), "init launch");
}

uint32_t iteration_grid(const Staged& g, uint32_t k, bool all_levels) {
    const uint32_t iso = k <= 2 || all_levels ? ceil_div(g.n_iso, kIsoPerBlock) : 0u;
    return std::max<uint32_t>(g.n_hub_chunks + g.n_solo + iso + ceil_div(g.n_tiles, kWaves), 1);
}

static SplitArgs split_args(const Staged& g, const RunBuffers& rb, uint32_t k) {
    SplitArgs a{};
    a.h = rb.h[k & 1];
    a.rep = rb.rep;
    a.act = g.act;
    a.solo_v = g.solo_v;
    a.hub_v = g.hub_v;
    a.n_act = g.n_act;
    a.n_solo = g.n_solo;
    a.count = k == 1 ? g.n : g.n_act + g.n_solo + g.n_hubs;
    a.test_tab = rb.tab[k & 1];
    a.clr_tab = rb.tab[(k - 1) & 1];
    a.lcnt = rb.lcnt;
    a.status = rb.status;
    a.k = k;
    a.bc = rb.bc;
    return a;
}

static uint32_t split_grid(const SplitArgs& a) {
    return std::max<uint32_t>(ceil_div(a.count, kBlock * kSplitPerThread), 1);
}

void launch_iteration(const Staged& g, const RunBuffers& rb, uint32_t k, uint32_t lag, uint32_t k_max, bool stop,
                      bool all_levels, uint64_t* report, IterParts parts, hipStream_t s) {
    IterArgs a{};
    a.stop_only = parts == IterParts::kStopTest ? 1u : 0u;
    a.report = report;
    a.lag = lag;
    a.row_off = g.row_off;
    a.tgt = g.tgt;
    a.lab = g.lab;
    a.t = rb.t;
    a.salt = g.salt;
    a.h_prev = rb.h[(k - 1) & 1];
    a.h_next = rb.h[k & 1];
    a.alive = g.alive;
    a.tiles = g.tiles;
    a.act = g.act;
    a.act_off = g.act_off;
    a.m = g.m;
    a.iso = g.iso;
    a.n_iso = g.n_iso;
    a.n_iso_blocks = k <= 2 || all_levels ? ceil_div(g.n_iso, kIsoPerBlock) : 0u;
    a.hc_hub = g.hc_hub;
    a.hc_e0 = g.hc_e0;
    a.hub_v = g.hub_v;
    a.hub_logb = g.hub_logb;
    a.hub_key_off = g.hub_key_off;
    a.hub_keys = rb.hub_keys;
    a.hub_boff = rb.hub_boff;
    a.lcnt = rb.lcnt;
    a.totals = rb.totals;
    a.status = rb.status;
    a.n_tiles = g.n_tiles;
    a.n_hub_chunks = g.n_hub_chunks;
    a.n_solo = g.n_solo;
    a.solo_v = g.solo_v;
    a.k = k;
    a.k_max = k_max;
    a.stop = stop ? 1u : 0u;
    a.bc = rb.bc;
    if (parts == IterParts::kHashesAndSplit || parts == IterParts::kSplit) {
        const SplitArgs sp = split_args(g, rb, k - 1);
        const uint32_t n_hash = parts == IterParts::kSplit ? 0u : iteration_grid(g, k, all_levels);
        const uint32_t grid = n_hash + split_grid(sp);
        if (g.label_bytes == 2)
            k_iterate_split<uint16_t><<<grid, kBlock, 0, s>>>(a, sp, n_hash);
        else
            k_iterate_split<uint32_t><<<grid, kBlock, 0, s>>>(a, sp, n_hash);
    } else {
        const uint32_t grid = parts == IterParts::kStopTest ? 1u : iteration_grid(g, k, all_levels);
        if (g.label_bytes == 2)
            k_iterate<uint16_t><<<grid, kBlock, 0, s>>>(a);
        else
            k_iterate<uint32_t><<<grid, kBlock, 0, s>>>(a);
    }
    hip_check(hipGetLastError(), "iteration launch");
}

void launch_split(const Staged& g, const RunBuffers& rb, uint32_t k, hipStream_t s) {
    const SplitArgs a = split_args(g, rb, k);
    k_split<<<split_grid(a), kBlock, 0, s>>>(a);
    hip_check(hipGetLastError(), "split launch");
}

void launch_hubs(const Staged& g, const RunBuffers& rb, uint32_t k, hipStream_t s) {
    if (g.n_hub_blocks == 0) return;
    HubArgs a{};
    a.t = rb.t;
    a.hub_keys = rb.hub_keys;
    a.hub_key_off = g.hub_key_off;
    a.hub_boff = rb.hub_boff;
    a.hub_chunk0 = g.hub_chunk0;
    a.hub_nchunks = g.hub_nchunks;
    a.hc_e0 = g.hc_e0;
    a.hub_v = g.hub_v;
    a.hub_logb = g.hub_logb;
    a.hb_hub = g.hb_hub;
    a.hb_bucket = g.hb_bucket;
    a.hub_acc = rb.hub_acc;
    a.h_next = rb.h[k & 1];
    a.status = rb.status;
    a.table_slots = g.hub_table_slots;
    a.table_limit = (g.hub_table_slots / 8) * 7;
    a.k = k;
    a.bc = rb.bc;
    k_hub<<<g.n_hub_blocks, kHubBlock, static_cast<size_t>(g.hub_table_slots) * 8, s>>>(a);
    hip_check(hipGetLastError(), "hub launch");
}

void alloc_hash_scratch(const Staged& g, HashScratch& hs, Arena& arena, hipStream_t s) {
    hs.hub_keys = arena.alloc<uint64_t>(g.hub_keys_total + 1);
    hs.hub_boff = arena.alloc<uint32_t>((static_cast<size_t>(g.n_hub_chunks) + 1) * kHubOffStride);
    hs.hub_acc = arena.alloc<uint64_t>(2ull * g.n_hubs + 2);
    hs.status = arena.alloc<RunStatus>(1);
    hip_check(hipMemsetAsync(hs.hub_acc, 0, (g.n_hubs + 1) * 16ull, s), "hub acc");
    hip_check(hipMemsetAsync(hs.status, 0, sizeof(RunStatus), s), "status");
}

void launch_hash_level(const Staged& g, const uint64_t* t, const uint64_t* h_prev, uint64_t* h_next,
                       const HashScratch& hs, uint32_t level, hipStream_t s) {
    IterArgs a{};
    a.row_off = g.row_off;
    a.tgt = g.tgt;
    a.lab = g.lab;
    a.t = t;
    a.salt = g.salt;
    a.h_prev = h_prev;
    a.h_next = h_next;
    a.alive = g.alive;
    a.tiles = g.tiles;
    a.act = g.act;
    a.act_off = g.act_off;
    a.m = g.m;
    a.iso = g.iso;
    a.n_iso = g.n_iso;
    a.n_iso_blocks = ceil_div(g.n_iso, kIsoPerBlock);
    a.hc_hub = g.hc_hub;
    a.hc_e0 = g.hc_e0;
    a.hub_v = g.hub_v;
    a.hub_logb = g.hub_logb;
    a.hub_key_off = g.hub_key_off;
    a.hub_keys = hs.hub_keys;
    a.hub_boff = hs.hub_boff;
    a.status = hs.status;
    a.n_tiles = g.n_tiles;
    a.n_hub_chunks = g.n_hub_chunks;
    a.n_solo = g.n_solo;
    a.solo_v = g.solo_v;
    a.k = level;
    a.k_max = 0xFFFFFFFFu;
    a.hash_only = 1;
    const uint32_t grid = iteration_grid(g, level, true);
    if (g.label_bytes == 2)
        k_iterate<uint16_t><<<grid, kBlock, 0, s>>>(a);
    else
        k_iterate<uint32_t><<<grid, kBlock, 0, s>>>(a);
    hip_check(hipGetLastError(), "hash level launch");
    if (g.n_hub_blocks == 0) return;
    HubArgs h{};
    h.t = t;
    h.hub_keys = hs.hub_keys;
    h.hub_key_off = g.hub_key_off;
    h.hub_boff = hs.hub_boff;
    h.hub_chunk0 = g.hub_chunk0;
    h.hub_nchunks = g.hub_nchunks;
    h.hc_e0 = g.hc_e0;
    h.hub_v = g.hub_v;
    h.hub_logb = g.hub_logb;
    h.hb_hub = g.hb_hub;
    h.hb_bucket = g.hb_bucket;
    h.hub_acc = hs.hub_acc;
    h.h_next = h_next;
    h.status = hs.status;
    h.table_slots = g.hub_table_slots;
    h.table_limit = (g.hub_table_slots / 8) * 7;
    h.k = level;
    k_hub<<<g.n_hub_blocks, kHubBlock, static_cast<size_t>(g.hub_table_slots) * 8, s>>>(h);
    hip_check(hipGetLastError(), "hash level hub launch");
}

void launch_graph_stop(const RunBuffers& rb, uint32_t k, uint32_t lag, uint32_t k_max, bool stop, hipStream_t s) {
    k_graph_stop<<<ceil_div(rb.bc.n_graphs, kBlock), kBlock, 0, s>>>(rb.bc, k, lag, k_max, stop ? 1u : 0u, rb.status);
    hip_check(hipGetLastError(), "graph stop launch");
}

}  // namespace bsim

// bsim_final.hip -- finalize (a8): relabel the final hashes to dense block
// ids, count block sizes, and build the summary graph's edges.
//
// Algorithm 4 ends with FindAndMerge: vertices with equal final identifiers
// form one block.  The refinement loop already names every vertex's class
// by a representative member; block ids are numbered by first occurrence
// (the block of the smallest vertex is 0), which depends only on the
// partition:
//   1. the smallest vertex of each class (atomicMin per class);
//   2. a bit per vertex "v is its class's smallest vertex", counted per
//      workgroup; an exclusive scan of the counts gives every such vertex its
//      block id, which it leaves under its class's name;
//   3. every vertex takes the id under its class's name; the members besides
//      the smallest are counted per workgroup in LDS first.
// Summary edges (Sec. 2.6: edges between vertex summaries) are the distinct
// (block(v), l, block(w)) triples.  Graphs with a tile schedule take them from
// bsim_sedges.hip; a resident state, which keeps its edges as (source, label,
// target) lists, packs one 64-bit key per edge here, sorts the keys by an LSD
// radix sort over the used bits, and unpacks the distinct ones.
#include "bsim_api_internal.h"
#include "bsim_device.h"

namespace bsim {

namespace {

// Smallest vertex of every class.  Classes are named by a member vertex
// (kOwn: cmin starts as the identity, and only vertices below their
// representative can lower it) or by a slot of a class index (cmin starts at
// the largest value).  A class of millions of vertices would have every wave
// in flight lower the same word: the lanes of a wave that share a class send
// its smallest, for the first kMinRounds classes among them.  On the names of
// a resident state of 2^22 R-MAT vertices 480 us became 148, on 2^22 R-MAT
// vertices of a summary 252 us became 43.
constexpr int kMinRounds = 4;

// Class minima before k_fin_min: the name itself (own) or none.  The launch
// also clears the words that later launches of the call count in: three
// clears and the salts' launch fewer (those are in k_types now) took a call on
// 1,000 vertices and 5,000 edges from 362 to 350 us.
__global__ void __launch_bounds__(kBlock) k_fin_init(uint32_t* __restrict__ cmin, uint32_t n, bool own,
                                                     uint32_t* __restrict__ zero, uint32_t n_zero,
                                                     uint32_t* __restrict__ zero2, uint32_t n_zero2) {
    const uint32_t v = blockIdx.x * kBlock + threadIdx.x;
    if (v < n) cmin[v] = own ? v : 0xFFFFFFFFu;
    if (v < n_zero) zero[v] = 0;
    if (v < n_zero2) zero2[v] = 0;
}

template <bool kOwn>
__global__ void __launch_bounds__(kBlock) k_fin_min(const uint32_t* __restrict__ rep,
                                                    const uint8_t* __restrict__ alive, uint32_t n, uint32_t* cmin) {
    const uint32_t v = blockIdx.x * kBlock + threadIdx.x;
    bool pending = v < n && (!alive || alive[v]);
    const uint32_t r = pending ? rep[v] : 0u;
    if (kOwn) pending = pending && v < r;
    for (int round = 0; round < kMinRounds; round++) {
        const uint64_t ball = __ballot(pending);
        if (!ball) return;
        const uint32_t leader = static_cast<uint32_t>(__ffsll(static_cast<long long>(ball)) - 1);
        const uint32_t lr = static_cast<uint32_t>(__shfl(static_cast<int>(r), static_cast<int>(leader), 64));
        if (pending && r == lr) {
            // (the first lane holds the smallest vertex.)  The minimum only
            // decreases: nothing to do once it is below v, as the device sees
            // it now; a line of this CU's cache could show the first value
            // for as long as the kernel runs
            if (lane_id() == leader &&
                __hip_atomic_load(&cmin[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > v)
                atomicMin(&cmin[r], v);
            pending = false;
        }
    }
    if (pending && cmin[r] > v) atomicMin(&cmin[r], v);
}

// Workgroups of kIdsPerBlock vertices, a 64-bit word per 64 of them.
constexpr int kIdsPerThread = 8;
constexpr int kIdsPerBlock = kBlock * kIdsPerThread;
constexpr int kIdsWords = kIdsPerBlock / 64;
constexpr int kIdsSlots = 2 * kIdsPerBlock;

__global__ void __launch_bounds__(kBlock) k_fin_first(const uint32_t* __restrict__ rep,
                                                      const uint8_t* __restrict__ alive, uint32_t n,
                                                      const uint32_t* __restrict__ cmin,
                                                      uint64_t* __restrict__ first, uint32_t* __restrict__ count) {
    __shared__ uint32_t s_red[kBlock / 64];
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kIdsPerBlock;
    uint32_t c = 0;
#pragma unroll
    for (int r = 0; r < kIdsPerThread; r++) {
        const uint64_t v = base + r * kBlock + threadIdx.x;
        const bool is = v < n && (!alive || alive[v]) && cmin[rep[v]] == static_cast<uint32_t>(v);
        const uint64_t bal = __ballot(is);
        if (lane_id() == 0) first[static_cast<uint64_t>(blockIdx.x) * kIdsWords + r * kWaves + (threadIdx.x >> 6)] = bal;
        c += static_cast<uint32_t>(__popcll(bal));
    }
    if (lane_id() == 0) s_red[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kBlock / 64; i++) c += s_red[i];
        count[blockIdx.x] = c;
    }
}

// The block id of every class's smallest vertex, under the class's name
// (cmin is not read any more), and a size of one for the block.
__global__ void __launch_bounds__(kBlock) k_fin_name(const uint32_t* __restrict__ rep,
                                                     const uint64_t* __restrict__ first,
                                                     const uint32_t* __restrict__ start, uint32_t nb,
                                                     uint32_t* __restrict__ name, uint32_t* __restrict__ sizes) {
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kIdsPerBlock;
    const uint64_t* word = first + static_cast<uint64_t>(blockIdx.x) * kIdsWords;
    const uint32_t lane = lane_id();
    // vertices before each word's: one word per lane (kIdsWords <= 64)
    const uint32_t c = lane < static_cast<uint32_t>(kIdsWords) ? static_cast<uint32_t>(__popcll(word[lane])) : 0u;
    const uint32_t excl = wave_incl_sum(c) - c;
    const uint32_t id0 = start[blockIdx.x];
#pragma unroll
    for (int r = 0; r < kIdsPerThread; r++) {
        const uint32_t g = r * kWaves + (threadIdx.x >> 6);
        const uint64_t w = word[g];
        const uint32_t before = static_cast<uint32_t>(__shfl(static_cast<int>(excl), static_cast<int>(g), 64));
        if ((w >> lane) & 1) {
            const uint32_t id = block_slot(id0 + before + static_cast<uint32_t>(__popcll(w & ((1ull << lane) - 1))), nb);
            name[rep[base + r * kBlock + threadIdx.x]] = id;
            sizes[id] = 1;
        }
    }
}

// Block ids.  Members besides the smallest are counted in an LDS table per
// workgroup first, so a block holding millions of vertices costs one global
// atomic per workgroup rather than one per vertex; most blocks hold one
// vertex and cost none.
//
// Bound: rep and the ids streamed, the names gathered.  With a rank array
// gathered through the class minimum and every vertex counted, 2^24 uniform
// vertices took 669 us and 2^27 R-MAT vertices 5.5 ms; now 54 us and 3.2 ms
// (the naming pass adds 34 and 390 us).
__global__ void __launch_bounds__(kBlock) k_fin_ids(const uint8_t* __restrict__ alive, uint32_t n,
                                                    const uint32_t* __restrict__ rep,
                                                    const uint32_t* __restrict__ name,
                                                    const uint64_t* __restrict__ first, uint32_t nb,
                                                    uint32_t* __restrict__ block_ids, uint32_t* __restrict__ sizes) {
    __shared__ uint32_t s_key[kIdsSlots];
    __shared__ uint32_t s_cnt[kIdsSlots];
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kIdsPerBlock;
    const uint64_t* word = first + static_cast<uint64_t>(blockIdx.x) * kIdsWords;
    const uint32_t lane = lane_id();
    uint32_t bid[kIdsPerThread];
    uint32_t more = 0;  // bit r: a member to be counted
#pragma unroll
    for (int r = 0; r < kIdsPerThread; r++) {
        const uint64_t v = base + r * kBlock + threadIdx.x;
        bid[r] = 0xFFFFFFFFu;
        if (v < n && (!alive || alive[v])) {
            bid[r] = block_slot(name[rep[v]], nb);
            if (!((word[r * kWaves + (threadIdx.x >> 6)] >> lane) & 1)) more |= 1u << r;
        }
    }
#pragma unroll
    for (int r = 0; r < kIdsPerThread; r++) {
        const uint64_t v = base + r * kBlock + threadIdx.x;
        if (v < n) block_ids[v] = bid[r];
    }
    if (!__syncthreads_or(more != 0)) return;
    for (int i = threadIdx.x; i < kIdsSlots; i += kBlock) {
        s_key[i] = 0xFFFFFFFFu;
        s_cnt[i] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kIdsPerThread; r++) {
        if (!((more >> r) & 1)) continue;
        uint32_t slot = (bid[r] * 2654435761u) & (kIdsSlots - 1);
        for (;;) {
            uint32_t cur = s_key[slot];
            if (cur == 0xFFFFFFFFu) cur = atomicCAS(&s_key[slot], 0xFFFFFFFFu, bid[r]);
            if (cur == 0xFFFFFFFFu || cur == bid[r]) break;
            slot = (slot + 1) & (kIdsSlots - 1);
        }
        atomicAdd(&s_cnt[slot], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kIdsSlots; i += kBlock)
        if (s_cnt[i]) atomicAdd(&sizes[s_key[i]], s_cnt[i]);
}

// ------------------------------------------------------------ radix sort
//
// LSD radix sort of 64-bit keys, 8 bits per pass.  Each pass: per-block digit
// histograms (digit-major, so one exclusive scan yields every block's output
// offset per digit), then a stable scatter that ranks equal digits by wave
// ballots (8 ballots isolate the lanes with the same digit).

// 16 keys per thread: a tile of 4,096 keys leaves about 16 keys per digit
// run, so the scatter writes runs of about 128 bytes
constexpr int kSortItems = 16;
constexpr int kSortTile = kBlock * kSortItems;

// Edge keys from a source per edge (a resident state).
template <typename LabT>
__global__ void __launch_bounds__(kBlock) k_edge_keys_coo(const uint32_t* __restrict__ src,
                                                          const uint32_t* __restrict__ tgt,
                                                          const LabT* __restrict__ lab,
                                                          const uint32_t* __restrict__ bid,
                                                          const uint32_t* __restrict__ bid_dst, uint32_t m,
                                                          int lb, int bb, uint64_t* __restrict__ keys) {
    const uint32_t e = blockIdx.x * kBlock + threadIdx.x;
    if (e >= m) return;
    keys[e] = (static_cast<uint64_t>(bid[src[e]]) << (lb + bb)) |
              (static_cast<uint64_t>(lab[e]) << bb) | bid_dst[tgt[e]];
}

__global__ void __launch_bounds__(kBlock) k_sort_hist(const uint64_t* __restrict__ in, uint32_t m,
                                                      int shift, uint32_t nblk,
                                                      uint32_t* __restrict__ hist) {
    __shared__ uint32_t s_h[256];
    s_h[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kSortTile;
#pragma unroll
    for (int r = 0; r < kSortItems; r++) {
        uint64_t j = base + static_cast<uint64_t>(r) * kBlock + threadIdx.x;
        if (j < m) atomicAdd(&s_h[(in[j] >> shift) & 0xFF], 1u);
    }
    __syncthreads();
    hist[static_cast<uint64_t>(threadIdx.x) * nblk + blockIdx.x] = s_h[threadIdx.x];
}

// Stable scatter of one tile: every key gets its rank within the tile by
// digit (wave ballots isolate the lanes with the same digit; earlier rounds
// and earlier waves come first), the tile is staged in LDS in digit order,
// and each digit's run is then written out by consecutive threads.
__global__ void __launch_bounds__(kBlock) k_sort_scatter(const uint64_t* __restrict__ in,
                                                         uint64_t* __restrict__ out, uint32_t m,
                                                         int shift, uint32_t nblk,
                                                         const uint32_t* __restrict__ offs) {
    __shared__ uint64_t s_keys[kSortTile];
    __shared__ uint32_t s_run[256];     // global position of the tile's first key of each digit
    __shared__ uint32_t s_start[256];   // LDS position of the same key
    __shared__ uint32_t s_fill[256];    // keys of each digit placed so far
    __shared__ uint32_t s_cnt[kBlock / 64][256];
    const uint32_t tid = threadIdx.x, lane = lane_id(), wid = tid >> 6;
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kSortTile;
    const uint32_t count = static_cast<uint32_t>(min(static_cast<uint64_t>(kSortTile), m - base));
    // the tile's keys per digit, from the scanned digit-major histogram: the
    // next entry is the next block of the same digit, or the first block of
    // the next digit, and the last entry ends at m
    const uint64_t idx = static_cast<uint64_t>(tid) * nblk + blockIdx.x;
    const uint32_t run = offs[idx];
    const uint32_t next = idx + 1 < static_cast<uint64_t>(nblk) * 256 ? offs[idx + 1] : m;
    s_run[tid] = run;
    s_start[tid] = next - run;
    s_fill[tid] = 0;
    for (int w = 0; w < kBlock / 64; w++) s_cnt[w][tid] = 0;
    __syncthreads();
    // exclusive scan of the 256 digit counts (one per thread)
    for (uint32_t d = 1; d < 256; d <<= 1) {
        const uint32_t v = tid >= d ? s_start[tid - d] : 0;
        __syncthreads();
        s_start[tid] += v;
        __syncthreads();
    }
    const uint32_t incl = s_start[tid];
    __syncthreads();
    s_start[tid] = incl - (next - run);
    __syncthreads();
    for (int r = 0; r < kSortItems; r++) {
        const uint32_t jl = static_cast<uint32_t>(r) * kBlock + tid;
        const bool valid = jl < count;
        const uint64_t key = valid ? in[base + jl] : 0;
        const uint32_t dig = static_cast<uint32_t>((key >> shift) & 0xFF);
        uint64_t peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < 8; b++) {
            const uint64_t bal = __ballot((dig >> b) & 1);
            peers &= ((dig >> b) & 1) ? bal : ~bal;
        }
        const uint64_t below = peers & ((1ull << lane) - 1);
        const uint32_t rank = static_cast<uint32_t>(__popcll(below));
        if (valid && below == 0) s_cnt[wid][dig] = static_cast<uint32_t>(__popcll(peers));
        __syncthreads();
        if (valid) {
            uint32_t pos = s_start[dig] + s_fill[dig] + rank;
            for (uint32_t w = 0; w < wid; w++) pos += s_cnt[w][dig];
            if (pos < kSortTile) s_keys[pos] = key;
        }
        __syncthreads();
        uint32_t add = 0;
        for (int w = 0; w < kBlock / 64; w++) {
            add += s_cnt[w][tid];
            s_cnt[w][tid] = 0;
        }
        s_fill[tid] += add;
        __syncthreads();
    }
    for (uint32_t i = tid; i < count; i += kBlock) {
        const uint64_t key = s_keys[i];
        const uint32_t dig = static_cast<uint32_t>((key >> shift) & 0xFF);
        const uint32_t pos = s_run[dig] + (i - s_start[dig]);
        if (pos < m) out[pos] = key;
    }
}

__global__ void __launch_bounds__(kBlock) k_unique_flags(const uint64_t* __restrict__ keys, uint32_t m,
                                                         uint32_t* __restrict__ flag) {
    uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < m) flag[i] = (i == 0 || keys[i] != keys[i - 1]) ? 1u : 0u;
}

__global__ void __launch_bounds__(kBlock) k_unpack(const uint64_t* __restrict__ keys, uint32_t m,
                                                   const uint32_t* __restrict__ flag,
                                                   const uint32_t* __restrict__ pos, int lb, int bb,
                                                   uint32_t* __restrict__ s, uint32_t* __restrict__ l,
                                                   uint32_t* __restrict__ d) {
    uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= m || !flag[i]) return;
    const uint64_t k = keys[i];
    const uint32_t p = pos[i];
    s[p] = static_cast<uint32_t>(k >> (lb + bb));
    l[p] = static_cast<uint32_t>((k >> bb) & ((1ull << lb) - 1));
    d[p] = static_cast<uint32_t>(k & ((1ull << bb) - 1));
}

}  // namespace

// Sort m keys ascending on bits [lo, bits); returns the buffer holding the
// result (a or b).
uint64_t* radix_sort(uint64_t* a, uint64_t* b, uint32_t m, int bits, Arena& arena, hipStream_t s, int lo) {
    if (m <= 1) return a;
    const uint32_t nblk = ceil_div(m, kSortTile);
    uint32_t* hist = arena.alloc<uint32_t>(static_cast<size_t>(nblk) * 256);
    for (int shift = lo; shift < bits; shift += 8) {
        k_sort_hist<<<nblk, kBlock, 0, s>>>(a, m, shift, nblk, hist);
        scan_exclusive(hist, hist, nblk * 256, nullptr, arena, s);
        k_sort_scatter<<<nblk, kBlock, 0, s>>>(a, b, m, shift, nblk, hist);
        std::swap(a, b);
    }
    hip_check(hipGetLastError(), "radix sort launch");
    return a;
}

namespace {

// First-occurrence block ids of the nb classes named by `rep` into ids[n],
// the block sizes into sizes_preset or a new array of `arena`; *seen receives
// the number of classes found.  zero, zero2: words cleared on the way, also
// with no vertices.
void number_blocks(const Staged& g, const uint32_t* rep, uint32_t nb, uint32_t* ids, uint32_t** sizes_out,
                   uint32_t* seen, Arena& arena, hipStream_t s, uint32_t* sizes_preset = nullptr,
                   uint64_t n_ids = 0, uint32_t* zero = nullptr, uint32_t n_zero = 0, uint32_t* zero2 = nullptr,
                   uint32_t n_zero2 = 0) {
    const uint32_t n = g.n;
    // class names are vertex ids, or below n_ids when given
    const uint64_t names = n_ids ? n_ids : n;
    uint32_t* name = arena.alloc<uint32_t>(names + 1);
    const uint32_t gb = ceil_div(n, kIdsPerBlock);
    uint64_t* first = arena.alloc<uint64_t>(static_cast<size_t>(gb) * kIdsWords + 1);
    uint32_t* count = arena.alloc<uint32_t>(gb + 1ull);
    uint32_t* sizes = sizes_preset ? sizes_preset : arena.alloc<uint32_t>(nb + 1ull);
    *sizes_out = sizes;
    const uint64_t wide = std::max<uint64_t>({names, n_zero, n_zero2, 1});
    k_fin_init<<<ceil_div(wide, kBlock), kBlock, 0, s>>>(name, static_cast<uint32_t>(names), n_ids == 0, zero, n_zero,
                                                         zero2, n_zero2);
    hip_check(hipGetLastError(), "finalize launch");
    if (!n) return;
    const uint32_t gv = ceil_div(n, kBlock);
    if (n_ids)
        k_fin_min<false><<<gv, kBlock, 0, s>>>(rep, g.alive, n, name);
    else
        k_fin_min<true><<<gv, kBlock, 0, s>>>(rep, g.alive, n, name);
    k_fin_first<<<gb, kBlock, 0, s>>>(rep, g.alive, n, name, first, count);
    scan_exclusive(count, count, gb, seen, arena, s);
    k_fin_name<<<gb, kBlock, 0, s>>>(rep, first, count, nb, name, sizes);
    k_fin_ids<<<gb, kBlock, 0, s>>>(g.alive, n, rep, name, first, nb, ids, sizes);
    hip_check(hipGetLastError(), "finalize launch");
}

void finalize_edges(const Staged& g, const uint32_t* rep, const uint32_t* rep_prev, bool want_edges,
                    FinalOut& out, FinalHost* host, Arena& arena, Arena& keep, hipStream_t s, uint64_t n_ids);

// Block ids and sizes are numbered in the call's work memory and copied
// into the result's own arrays at the end: the kernels that count the sizes
// (atomics at random blocks) and gather the ids of the edges' targets ran
// 10-20 % slower on rmat27 when these arrays were result allocations of
// their own beside the work memory's other random-access arrays.
void finalize_impl(const Staged& g, const uint32_t* rep, const uint32_t* rep_prev, bool want_edges,
                   FinalOut& out, FinalHost* host, Arena& arena, Arena& keep, hipStream_t s, uint64_t n_ids = 0) {
    if (out.preset) {
        finalize_edges(g, rep, rep_prev, want_edges, out, host, arena, keep, s, n_ids);
        return;
    }
    uint32_t* ids = keep.alloc<uint32_t>(g.n);
    out.block_ids = arena.alloc<uint32_t>(g.n);
    finalize_edges(g, rep, rep_prev, want_edges, out, host, arena, keep, s, n_ids);
    uint32_t* sizes = keep.alloc<uint32_t>(out.n_blocks + 1ull);
    void* const dst[2] = {ids, sizes};
    const void* const src[2] = {out.block_ids, out.block_sizes};
    const size_t bytes[2] = {static_cast<size_t>(g.n) * 4, static_cast<size_t>(out.n_blocks) * 4};
    copy_ranges(dst, src, bytes, 2, s);
    out.block_ids = ids;
    out.block_sizes = sizes;
}

void finalize_edges(const Staged& g, const uint32_t* rep, const uint32_t* rep_prev, bool want_edges,
                    FinalOut& out, FinalHost* host, Arena& arena, Arena& keep, hipStream_t s, uint64_t n_ids) {
    const uint32_t n = g.n;
    const uint32_t nb = out.n_blocks;
    // the counts that come back to the host, together
    FinalHost* dev = arena.alloc<FinalHost>(1);
    // a summary edge's target end: the final blocks, or the blocks of the
    // previous level
    const uint32_t nb_dst = rep_prev ? out.n_prev_blocks : nb;
    const uint32_t nb_max = std::max(nb, nb_dst);
    const int bb = std::max(1, bit_width(nb_max ? nb_max - 1 : 0));
    const int lb = std::max(1, bit_width(g.max_label));
    const bool bucketed = want_edges && g.m && bucketed_summary_edges_fit(g, lb, bb);
    uint32_t* ecount = bucketed ? arena.alloc<uint32_t>(static_cast<size_t>(nb) + 1) : nullptr;
    number_blocks(g, rep, nb, out.block_ids, &out.block_sizes, dev->blocks, arena, s,
                  out.preset ? out.block_sizes : nullptr, n_ids, reinterpret_cast<uint32_t*>(dev),
                  sizeof(FinalHost) / 4, ecount, bucketed ? nb + 1 : 0u);
    const std::function<const FinalHost&()> fetch = [&]() -> const FinalHost& {
        hip_check(hipMemcpyAsync(host, dev, sizeof(FinalHost), hipMemcpyDeviceToHost, s), "finalize counts");
        hip_check(hipStreamSynchronize(s), "finalize counts");
        if (host->blocks[0] != nb)
            throw DeviceError{BSIM_E_DEVICE, "internal: class count mismatch in finalize"};
        return *host;
    };
    out.n_se = 0;
    if (!want_edges || g.m == 0) {
        fetch();
        if (!out.preset) {
            out.se_src = keep.alloc<uint32_t>(1);
            out.se_label = keep.alloc<uint32_t>(1);
            out.se_dst = keep.alloc<uint32_t>(1);
        }
        return;
    }
    const uint32_t* dst_ids = out.block_ids;
    if (rep_prev) {
        uint32_t* ids = arena.alloc<uint32_t>(n);
        uint32_t* sizes = nullptr;
        number_blocks(g, rep_prev, nb_dst, ids, &sizes, dev->prev_blocks, arena, s);
        dst_ids = ids;
    }
    if (bucketed) {
        bucketed_summary_edges(g, out.block_ids, nb, dst_ids, lb, bb, ecount, out, dev, fetch, arena, keep, s);
        if (rep_prev && host->prev_blocks[0] != nb_dst)
            throw DeviceError{BSIM_E_DEVICE, "internal: class count mismatch in finalize"};
        return;
    }
    // (labels are below 2^24, so graphs with a tile schedule that the bucketed
    // path refuses, for more than 46 value bits, are refused here too)
    if (2 * bb + lb > 64 || !g.src)
        throw DeviceError{BSIM_E_UNSUPPORTED, "summary-edge triple does not fit 64 bits"};
    const uint32_t m = static_cast<uint32_t>(g.m);
    uint64_t* ka = arena.alloc<uint64_t>(m);
    uint64_t* kb = arena.alloc<uint64_t>(m);
    if (g.label_bytes == 2)
        k_edge_keys_coo<uint16_t><<<ceil_div(m, kBlock), kBlock, 0, s>>>(
            g.src, g.tgt, static_cast<const uint16_t*>(g.lab), out.block_ids, dst_ids, m, lb, bb, ka);
    else
        k_edge_keys_coo<uint32_t><<<ceil_div(m, kBlock), kBlock, 0, s>>>(
            g.src, g.tgt, static_cast<const uint32_t*>(g.lab), out.block_ids, dst_ids, m, lb, bb, ka);
    hip_check(hipGetLastError(), "edge key launch");
    uint64_t* sorted = radix_sort(ka, kb, m, 2 * bb + lb, arena, s);
    uint32_t* flag = arena.alloc<uint32_t>(m);
    uint32_t* pos = arena.alloc<uint32_t>(m);
    k_unique_flags<<<ceil_div(m, kBlock), kBlock, 0, s>>>(sorted, m, flag);
    scan_exclusive(flag, pos, m, dev->edges, arena, s);
    fetch();
    if (rep_prev && host->prev_blocks[0] != nb_dst)
        throw DeviceError{BSIM_E_DEVICE, "internal: class count mismatch in finalize"};
    const uint32_t nse = host->edges[0];
    out.n_se = nse;
    if (!out.preset) {
        out.se_src = keep.alloc<uint32_t>(nse);
        out.se_label = keep.alloc<uint32_t>(nse);
        out.se_dst = keep.alloc<uint32_t>(nse);
    }
    k_unpack<<<ceil_div(m, kBlock), kBlock, 0, s>>>(sorted, m, flag, pos, lb, bb, out.se_src,
                                                    out.se_label, out.se_dst);
    hip_check(hipGetLastError(), "unpack launch");
}

}  // namespace

void finalize(const Staged& g, const uint32_t* rep, bool want_edges, FinalOut& out, FinalHost* host, Arena& arena,
              Arena& keep, hipStream_t s, uint64_t n_ids) {
    finalize_impl(g, rep, nullptr, want_edges, out, host, arena, keep, s, n_ids);
}

void finalize_prev_level(const Staged& g, const uint32_t* rep, const uint32_t* rep_prev, bool want_edges,
                         FinalOut& out, FinalHost* host, Arena& arena, Arena& keep, hipStream_t s) {
    finalize_impl(g, rep, rep_prev, want_edges, out, host, arena, keep, s);
}

}  // namespace bsim

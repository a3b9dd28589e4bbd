// bsim_sedges.hip -- the summary graph's edges (a8), bucketed by source block.
//
// The summary edges (Sec. 2.6: edges between vertex summaries) are the
// distinct triples (block(v), l, block(w)) over the edges (v, l, w), listed
// by source block, then label, then target block.  A global sort of all m
// triples would move every edge through eight radix passes; here the edges
// are bucketed by source block first, so only the (label, target block)
// values inside one block's segment are ever compared:
//   1. every vertex with out-edges claims a range of its block's segment
//      (one atomic per vertex); an exclusive scan over the blocks places
//      the segments;
//   2. every edge writes its value l << bb | block(w) into its vertex's range;
//   3. every segment is sorted and de-duplicated in place, by size:
//        1 value          nothing to do;
//        2..128           one wave takes the segments starting in 256
//                         consecutive positions; every value counts the ones
//                         of its segment up to it;
//        129..16,384      one wave (up to 512 values) or workgroup per segment (of
//                         512 threads up to 4,096 values, else 1,024): the
//                         values go to buckets by their highest bits that
//                         differ, and each counts the ones of its bucket up
//                         to it; LDS radix sort where that would read more,
//                         and for the largest class;
//        more             one global LSD radix sort over all such segments
//                         on (segment rank, value);
//   4. an exclusive scan of the per-block distinct counts places the output;
//      the distinct values are unpacked to (src, label, dst).
// Repeated values end at one place, and the value found there last is kept.
#include "bsim_device.h"

namespace bsim {

namespace {

constexpr uint32_t kSegSmallMax = 128;     // tile-packed segments hold at most this many values
constexpr uint32_t kSegMidMax = 512;       // one wave per segment
constexpr uint32_t kMedBlock = 512;
constexpr uint32_t kMedWaves = kMedBlock / 64;
constexpr uint32_t kSegMedMax = 4096;      // one workgroup of kMedBlock per segment
constexpr uint32_t kBigBlock = 1024;
constexpr uint32_t kSegBigMax = 16384;     // one workgroup of kBigBlock per segment
constexpr uint32_t kSmallBlock = 64;       // a small tile is one wave
constexpr uint32_t kSmallRange = 256;      // segment starts per small tile
constexpr uint32_t kSmallCap = 384;        // values per small tile
constexpr uint32_t kSmallRounds = kSmallCap / kSmallBlock;   // values per lane
constexpr uint32_t kSmallMaxSeg = kSmallRange / 2;           // segments of >= 2 values
// Segments of the wave class above which they get a launch of their own, where
// more of their waves fit a CU; fewer do not fill the chip, and wait less
// beside the longer ones (2^20 edges: 34 + 40 us for two launches, 28 for one).
constexpr uint32_t kMidApart = 4096;
// A value counts the ones of its bucket, so a segment costs the squares of its
// bucket lengths in reads; a radix pass costs each value about kRankReads of
// them, and there is one per byte in which the values differ.  A limit on the
// longest bucket instead (512) let segments of 600 values in two buckets of 300
// through at many times the cost of their two passes.  2^25 edges in segments of
// 8 (1,024) distinct values, whole call, 600 values a segment: 2.73 (1.66) ms
// with that limit, 1.67 (1.65) with 24 reads, 1.67 (1.93) with 12 and 1.69
// (1.65) with 96; 500 values: 2.07 (2.13), 1.15 (1.36), 1.15 (1.37) and 1.16
// (2.15).  R-MAT graphs take the same with any of these.
constexpr uint32_t kRankReads = 24;
constexpr uint32_t kUnpackTile = kBlock * 16;
constexpr uint32_t kUnpackCache = 4096;    // block offsets a tile keeps in LDS

static_assert(kSmallRange + kSegSmallMax - 1 <= kSmallCap, "a small tile must hold its segments");

// A segment is sorted by a group of NT threads: one wave of a workgroup
// (NT = 64), or the workgroup.
template <int NT>
__device__ __forceinline__ uint32_t group_tid() { return NT == 64 ? lane_id() : threadIdx.x; }

template <int NT>
__device__ __forceinline__ void group_sync() {
    if constexpr (NT == 64)
        wave_sync();
    else
        __syncthreads();
}

// Exclusive scan over the group; *total gets the sum.  All threads must call
// it.  `red` needs NT / 64 entries.
template <int NT>
__device__ __forceinline__ uint32_t group_excl_scan(uint32_t x, uint32_t* red, uint32_t* total) {
    const uint32_t incl = wave_incl_sum(x);
    if constexpr (NT == 64) {
        *total = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), 63));
        return incl - x;
    }
    const uint32_t w = threadIdx.x >> 6;
    if (lane_id() == 63) red[w] = incl;
    __syncthreads();
    uint32_t base = 0, tot = 0;
    for (uint32_t i = 0; i < NT / 64; i++) {
        const uint32_t r = red[i];
        if (i < w) base += r;
        tot += r;
    }
    __syncthreads();
    *total = tot;
    return base + incl - x;
}

// Position of the last entry of off[lo, hi) that is <= x (off nondecreasing,
// off[lo] <= x).
__device__ __forceinline__ uint32_t last_le(const uint32_t* off, uint32_t lo, uint32_t hi, uint32_t x) {
    while (hi - lo > 1) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (off[mid] <= x)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// LDS of one segment's sort.  The largest class fills a CU's memory with its
// keys and counters and is sorted by radix passes alone.
constexpr uint16_t kNoMark = 0xFFFF;
template <int NT>
struct SegSmem {
    static constexpr bool kBucketed = NT < kBigBlock;
    static constexpr uint32_t kCap = NT == 64 ? kSegMidMax : NT == kMedBlock ? kSegMedMax : kSegBigMax;
    static constexpr uint32_t kIpt = kCap / NT;  // keys per thread
    static constexpr uint32_t kCounters = NT == 64 ? 512 : NT * 4;  // (a radix pass needs 256 a wave)
    uint64_t* buf;   // [kCap] keys
    uint32_t* wc;    // [kCounters] bucket bounds, or a digit's counters per wave
    uint32_t* red;   // [16]
    uint16_t* mark;  // [kCap] which key has each place, kNoMark where none has
    __device__ explicit SegSmem(uint64_t* p)
        : buf(p), wc(reinterpret_cast<uint32_t*>(p + kCap)), red(wc + kCounters),
          mark(reinterpret_cast<uint16_t*>(red + 16)) {}
    static constexpr uint64_t bytes() { return (kBucketed ? 10ull : 8ull) * kCap + 4ull * kCounters + 4 * 16; }
};

struct SegArgs {
    uint64_t* vals;             // bucketed values, sorted and compacted in place
    const uint32_t* estart;     // nb + 1 segment offsets (estart[nb] = live edges)
    uint32_t nb;
    uint32_t* uniq;             // distinct values per block
    const uint32_t* tile_first; // small tiles: first block whose segment starts in the tile
    uint32_t n_tiles;
    const uint32_t *l_mid, *l_med, *l_big;   // longer segments by class: their blocks
    const uint32_t *n_mid, *n_med, *n_big;   // and their number
    int vb;                     // value bits
};

// The differing bits of the group's keys (kor, kand: a thread's own).
template <int NT>
__device__ uint64_t differing_bits(const SegSmem<NT>& S, uint64_t kor, uint64_t kand) {
    constexpr uint32_t W = NT / 64;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        kor |= shfl_xor_u64(kor, d);
        kand &= shfl_xor_u64(kand, d);
    }
    if (lane_id() == 0) {
        S.buf[2 * (group_tid<NT>() >> 6)] = kor;
        S.buf[2 * (group_tid<NT>() >> 6) + 1] = kand;
    }
    group_sync<NT>();
    uint64_t o = 0, n = ~0ull;
    for (uint32_t i = 0; i < W; i++) {
        o |= S.buf[2 * i];
        n &= S.buf[2 * i + 1];
    }
    group_sync<NT>();
    return o ^ n;
}

// Sort the segment's cnt keys by radix passes over the digits with differing
// bits: digits are ranked with wave ballots into per-wave counters.  key[r]
// is element (w * ipt + r) * 64 + lane, before and after (~0 past the end).
template <int NT>
__device__ void radix_segment(const SegSmem<NT>& S, uint32_t cnt, uint32_t ipt, uint64_t diff,
                              uint64_t (&key)[SegSmem<NT>::kIpt]) {
    constexpr uint32_t W = NT / 64;
    constexpr uint32_t DPT = NT >= 256 ? 1 : 256 / NT;  // digits per thread in the prefix step
    const uint32_t tid = group_tid<NT>(), lane = lane_id(), w = tid >> 6;
    const uint64_t lt = (1ull << lane) - 1;
    constexpr uint32_t kIpt = SegSmem<NT>::kIpt;
    uint32_t lr[kIpt];
    for (int shift = 0; shift < 64; shift += 8) {
        if (((diff >> shift) & 0xFF) == 0) continue;  // uniform over the group
        for (uint32_t d = lane; d < 256; d += 64) S.wc[w * 256 + d] = 0;
        wave_sync();
        // wave-local stable ranks per digit
#pragma unroll
        for (uint32_t r = 0; r < kIpt; r++) {
            if (r >= ipt) continue;
            const uint32_t i = (w * ipt + r) * 64 + lane;
            const bool valid = i < cnt;
            const uint32_t dig = static_cast<uint32_t>((key[r] >> shift) & 0xFF);
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 8; b++) {
                const uint64_t bal = __ballot((dig >> b) & 1);
                peers &= ((dig >> b) & 1) ? bal : ~bal;
            }
            const uint32_t leader = peers ? static_cast<uint32_t>(__ffsll(static_cast<long long>(peers)) - 1) : lane;
            uint32_t base = 0;
            if (valid && lane == leader) base = atomicAdd(&S.wc[w * 256 + dig], static_cast<uint32_t>(__popcll(peers)));
            base = static_cast<uint32_t>(__shfl(static_cast<int>(base), static_cast<int>(leader), 64));
            lr[r] = base + static_cast<uint32_t>(__popcll(peers & lt));
        }
        group_sync<NT>();
        // digit d of wave w starts at (keys of smaller digits) + (digit d in
        // earlier waves); thread t owns digits [t DPT, (t + 1) DPT)
        const bool owner = tid * DPT < 256;
        uint32_t tot = 0;
        if (owner)
            for (uint32_t c = 0; c < DPT; c++)
                for (uint32_t i = 0; i < W; i++) tot += S.wc[i * 256 + tid * DPT + c];
        uint32_t all = 0;
        uint32_t run = group_excl_scan<NT>(owner ? tot : 0u, S.red, &all);
        if (owner)
            for (uint32_t c = 0; c < DPT; c++)
                for (uint32_t i = 0; i < W; i++) {
                    const uint32_t d = tid * DPT + c;
                    const uint32_t cc = S.wc[i * 256 + d];
                    S.wc[i * 256 + d] = run;
                    run += cc;
                }
        group_sync<NT>();
#pragma unroll
        for (uint32_t r = 0; r < kIpt; r++) {
            if (r >= ipt) continue;
            const uint32_t i = (w * ipt + r) * 64 + lane;
            if (i < cnt) {
                const uint32_t dig = static_cast<uint32_t>((key[r] >> shift) & 0xFF);
                S.buf[S.wc[w * 256 + dig] + lr[r]] = key[r];
            }
        }
        group_sync<NT>();
#pragma unroll
        for (uint32_t r = 0; r < kIpt; r++) {
            if (r >= ipt) continue;
            const uint32_t i = (w * ipt + r) * 64 + lane;
            if (i < cnt) key[r] = S.buf[i];
        }
    }
}

// LDS of a small tile.
struct SmallSmem {
    uint64_t val[kSmallCap + 4];       // the values, then the places
    uint8_t own[kSmallCap];            // segment of each value
    uint32_t lofs[kSmallMaxSeg + 1];   // first position of each segment in the tile
    uint32_t blk[kSmallMaxSeg];        // its block
    uint32_t est[kSmallMaxSeg];        // its first value in vals[]
};

// A value's place in its segment is the number of values up to it, so it reads
// its segment once from LDS (lanes of one segment read one address).  Equal
// values get one place; the one whose number is found there after all have
// written is kept, and the places taken before it are its rank.
template <typename V>
__device__ void rank_tile(const SegArgs& a, SmallSmem& S, uint32_t cnt, uint32_t nseg) {
    const uint32_t lane = lane_id();
    V* val = reinterpret_cast<V*>(S.val);
    for (uint32_t o = lane; o < nseg; o += 64)
        for (uint32_t i = S.lofs[o]; i < S.lofs[o + 1]; i++) S.own[i] = static_cast<uint8_t>(o);
    wave_sync();
    V x[kSmallRounds];
    uint32_t seg[kSmallRounds];  // first position << 16 | length
    uint32_t to[kSmallRounds];   // where the segment starts in vals
#pragma unroll
    for (uint32_t r = 0; r < kSmallRounds; r++) {
        const uint32_t i = r * 64 + lane;
        x[r] = 0;
        seg[r] = to[r] = 0;
        if (i < cnt) {
            const uint32_t o = S.own[i], s0 = S.lofs[o];
            seg[r] = s0 << 16 | (S.lofs[o + 1] - s0);
            to[r] = S.est[o];
            x[r] = static_cast<V>(a.vals[to[r] + (i - s0)]);
        }
    }
#pragma unroll
    for (uint32_t r = 0; r < kSmallRounds; r++)
        if (r * 64 + lane < cnt) val[r * 64 + lane] = x[r];
    wave_sync();
    uint32_t at[kSmallRounds];  // place of the value in the tile
#pragma unroll
    for (uint32_t r = 0; r < kSmallRounds; r++) {
        if (r * 64 >= cnt) continue;  // uniform
        const uint32_t s0 = seg[r] >> 16, len = seg[r] & 0xFFFF;
        uint32_t upto = 0;
        for (uint32_t j = 0; j < len; j += 4) {
            // (up to three reads past the segment stay inside the LDS block)
#pragma unroll
            for (uint32_t k = 0; k < 4; k++) upto += (val[s0 + j + k] <= x[r]) & (j + k < len);
        }
        at[r] = s0 + upto - 1;
    }
    wave_sync();
    // the values are in registers: their place now holds who wrote there
    uint16_t* mark = reinterpret_cast<uint16_t*>(S.val);
    uint16_t* before = mark + kSmallCap;
#pragma unroll
    for (uint32_t r = 0; r < kSmallRounds; r++) mark[r * 64 + lane] = 0xFFFF;
    wave_sync();
#pragma unroll
    for (uint32_t r = 0; r < kSmallRounds; r++)
        if (r * 64 + lane < cnt) mark[at[r]] = static_cast<uint16_t>(r * 64 + lane);
    wave_sync();
    uint32_t kept = 0;
    bool all = true;
#pragma unroll
    for (uint32_t r = 0; r < kSmallRounds; r++) {
        const uint32_t i = r * 64 + lane;
        const bool mine = i < cnt && mark[at[r]] == i;
        kept |= static_cast<uint32_t>(mine) << r;
        all = all && (mine || i >= cnt);
    }
    if (__all(all)) {
#pragma unroll
        for (uint32_t r = 0; r < kSmallRounds; r++)
            if (r * 64 + lane < cnt) a.vals[to[r] + at[r] - (seg[r] >> 16)] = x[r];
        for (uint32_t o = lane; o < nseg; o += 64) a.uniq[S.blk[o]] = S.lofs[o + 1] - S.lofs[o];
        return;
    }
    // before[p]: taken places below p
    uint32_t run = 0;
    const uint64_t lt = (1ull << lane) - 1;
#pragma unroll
    for (uint32_t r = 0; r < kSmallRounds; r++) {
        const uint64_t bal = __ballot(mark[r * 64 + lane] != 0xFFFF);
        before[r * 64 + lane] = static_cast<uint16_t>(run + static_cast<uint32_t>(__popcll(bal & lt)));
        run += static_cast<uint32_t>(__popcll(bal));
    }
    if (lane == 0) before[kSmallCap] = static_cast<uint16_t>(run);
    wave_sync();
#pragma unroll
    for (uint32_t r = 0; r < kSmallRounds; r++)
        if ((kept >> r) & 1) a.vals[to[r] + before[at[r]] - before[seg[r] >> 16]] = x[r];
    for (uint32_t o = lane; o < nseg; o += 64) a.uniq[S.blk[o]] = before[S.lofs[o + 1]] - before[S.lofs[o]];
}

// Small segments (2..128 values): tile t takes the small segments whose
// first value lies in [t R, (t + 1) R), R = kSmallRange, and packs them back
// to back.  A tile is one wave with 5 KB of LDS, so many share a CU.
//
// Counting reads a value's whole segment, a radix sort takes some five passes
// of eight ballots a value whatever the length: with radix the 2^27 values of
// a uniform graph (8 a segment) took 3.2 ms.  Counted beside a radix sort for
// tiles with a segment of 129 to 256 values they took 1.06 ms, and 1.17 (9.6)
// ms on R-MAT graphs of 2^24 (2^27) vertices, 1.56 where those were counted
// too; with those segments in a class of their own 0.70 and 0.46 (4.1).
__global__ void __launch_bounds__(kSmallBlock) k_seg_small(SegArgs a) {
    __shared__ SmallSmem S;
    const uint32_t t = blockIdx.x;
    const uint32_t b_lo = a.tile_first[t];
    const uint32_t b_hi = t + 1 < a.n_tiles ? a.tile_first[t + 1] : a.nb;
    uint32_t nseg = 0, cnt = 0;
    for (uint32_t c = b_lo; c < b_hi; c += kSmallBlock) {  // uniform trip count
        const uint32_t b = c + threadIdx.x;
        uint32_t sz = 0, e0 = 0;
        if (b < b_hi) {
            e0 = a.estart[b];
            sz = a.estart[b + 1] - e0;
        }
        const bool small = sz >= 2 && sz <= kSegSmallMax;
        const uint32_t mine = small ? (1u << 20) | sz : 0u;
        const uint32_t incl = wave_incl_sum(mine);
        const uint32_t tot = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(incl), 63));
        if (small) {
            const uint32_t packed = incl - mine;
            const uint32_t o = nseg + (packed >> 20);
            S.lofs[o] = cnt + (packed & 0xFFFFF);
            S.blk[o] = b;
            S.est[o] = e0;
        }
        nseg += tot >> 20;
        cnt += tot & 0xFFFFF;
    }
    if (nseg == 0) return;  // uniform
    if (threadIdx.x == 0) S.lofs[nseg] = cnt;
    wave_sync();
    if (a.vb <= 32)
        rank_tile<uint32_t>(a, S, cnt, nseg);
    else
        rank_tile<uint64_t>(a, S, cnt, nseg);
}

// Places of a segment's keys by counting: to buckets by their highest
// differing bits, then each key counts the ones of its bucket up to it.  On
// return S.mark holds a key per taken place, S.buf the keys; false where that
// reads more than radix passes cost (S.buf and S.wc are free again).
template <int NT>
__device__ bool rank_segment(const SegSmem<NT>& S, uint32_t cnt, uint32_t ipt, uint64_t diff,
                             const uint64_t (&key)[SegSmem<NT>::kIpt]) {
    constexpr uint32_t kIpt = SegSmem<NT>::kIpt;
    constexpr uint32_t kBuckets = SegSmem<NT>::kCounters;
    constexpr int kBucketBits = NT == 64 ? 9 : 11;
    constexpr uint32_t kOwn = kBuckets / NT / 4;  // groups of four buckets a thread counts
    static_assert(kBuckets == 1u << kBucketBits, "one bucket per digit");
    const uint32_t tid = group_tid<NT>(), lane = lane_id(), w = tid >> 6;
    const int top = 64 - __clzll(static_cast<long long>(diff));
    const int shift = top > kBucketBits ? top - kBucketBits : 0;
    auto bucket = [&](uint64_t k) { return static_cast<uint32_t>(k >> shift) & (kBuckets - 1); };
    uint4* own = reinterpret_cast<uint4*>(S.wc) + kOwn * tid;
#pragma unroll
    for (uint32_t i = 0; i < kOwn; i++) own[i] = make_uint4(0, 0, 0, 0);
    group_sync<NT>();
#pragma unroll
    for (uint32_t r = 0; r < kIpt; r++)
        if (r < ipt && (w * ipt + r) * 64 + lane < cnt) atomicAdd(&S.wc[bucket(key[r])], 1u);
    group_sync<NT>();
    uint4 c[kOwn];
    uint32_t reads = 0, sum = 0;  // (at most kCap^2 reads)
#pragma unroll
    for (uint32_t i = 0; i < kOwn; i++) {
        c[i] = own[i];
        reads += c[i].x * c[i].x + c[i].y * c[i].y + c[i].z * c[i].z + c[i].w * c[i].w;
        sum += c[i].x + c[i].y + c[i].z + c[i].w;
    }
    reads = wave_sum_u32(reads);
    if (NT > 64 && lane == 0) S.red[8 + w] = reads;  // (the scan uses the first eight)
    uint32_t all = 0;
    uint32_t at = group_excl_scan<NT>(sum, S.red, &all);
#pragma unroll
    for (uint32_t i = 0; i < kOwn; i++) {
        own[i] = make_uint4(at, at + c[i].x, at + c[i].x + c[i].y, at + c[i].x + c[i].y + c[i].z);
        at += c[i].x + c[i].y + c[i].z + c[i].w;
    }
    if constexpr (NT > 64) {
        reads = 0;
        for (uint32_t i = 0; i < NT / 64; i++) reads += S.red[8 + i];
    }
    group_sync<NT>();
    uint32_t passes = 0;
    for (int b = 0; b < 64; b += 8) passes += (diff >> b & 0xFF) != 0;
    if (reads > kRankReads * passes * cnt) return false;
    // scattered, a bucket's counter holds its end
#pragma unroll
    for (uint32_t r = 0; r < kIpt; r++)
        if (r < ipt && (w * ipt + r) * 64 + lane < cnt) S.buf[atomicAdd(&S.wc[bucket(key[r])], 1u)] = key[r];
    for (uint32_t r = 0; r < ipt; r++) S.mark[(w * ipt + r) * 64 + lane] = kNoMark;
    group_sync<NT>();
    for (uint32_t r = 0; r < ipt; r++) {
        const uint32_t i = (w * ipt + r) * 64 + lane;
        if (i >= cnt) break;
        const uint64_t k = S.buf[i];
        const uint32_t d = bucket(k), s0 = d ? S.wc[d - 1] : 0u, len = S.wc[d] - s0;
        uint32_t upto = 0;
        for (uint32_t j = 0; j < len; j += 8) {
            // (up to seven reads past the bucket stay inside the LDS block)
#pragma unroll
            for (uint32_t q = 0; q < 8; q++) upto += (S.buf[s0 + j + q] <= k) & (j + q < len);
        }
        S.mark[s0 + upto - 1] = static_cast<uint16_t>(i);
    }
    group_sync<NT>();
    return true;
}

// One longer segment: the group's threads sort block b's.
template <int NT>
__device__ void sort_segment(const SegArgs& a, uint64_t* smem, uint32_t b) {
    const SegSmem<NT> S(smem);
    constexpr uint32_t kIpt = SegSmem<NT>::kIpt;
    const uint32_t e0 = a.estart[b], cnt = a.estart[b + 1] - e0;
    uint64_t* vals = a.vals + e0;
    const uint32_t tid = group_tid<NT>(), lane = lane_id(), w = tid >> 6;
    const uint32_t ipt = (cnt + NT - 1) / NT;  // rounds per wave; element = (w * ipt + r) * 64 + lane
    uint64_t key[kIpt];
    uint64_t kor = 0, kand = ~0ull;
#pragma unroll
    for (uint32_t r = 0; r < kIpt; r++) {
        key[r] = ~0ull;
        const uint32_t i = (w * ipt + r) * 64 + lane;
        if (r < ipt && i < cnt) {
            key[r] = vals[i];
            kor |= key[r];
            kand &= key[r];
        }
    }
    const uint64_t diff = differing_bits(S, kor, kand);
    if (diff == 0) {  // one value (uniform)
        if (tid == 0) {
            vals[0] = key[0];
            a.uniq[b] = 1;
        }
        return;
    }
    bool ranked = false;
    if constexpr (SegSmem<NT>::kBucketed) ranked = rank_segment<NT>(S, cnt, ipt, diff, key);
    if (!ranked) {
        radix_segment<NT>(S, cnt, ipt, diff, key);
#pragma unroll
        for (uint32_t r = 0; r < kIpt; r++) {
            const uint32_t i = (w * ipt + r) * 64 + lane;
            if (r < ipt && i < cnt) S.buf[i] = key[r];
        }
        group_sync<NT>();
    }
    // the key of place i if it is a distinct one's: the distinct values in order
    auto distinct_at = [&](uint32_t i) -> uint32_t {
        if (ranked) return S.mark[i];
        return i < cnt && (i == 0 || S.buf[i - 1] != S.buf[i]) ? i : kNoMark;
    };
    uint32_t mine = 0;
    for (uint32_t r = 0; r < ipt; r++)
        mine += static_cast<uint32_t>(__popcll(__ballot(distinct_at((w * ipt + r) * 64 + lane) != kNoMark)));
    if (lane == 0) S.red[w] = mine;
    group_sync<NT>();
    uint32_t at = 0, distinct = 0;
    for (uint32_t i = 0; i < NT / 64; i++) {
        if (i < w) at += S.red[i];
        distinct += S.red[i];
    }
    for (uint32_t r = 0; r < ipt; r++) {
        const uint32_t i = distinct_at((w * ipt + r) * 64 + lane);
        const uint64_t bal = __ballot(i != kNoMark);
        if (i != kNoMark) vals[at + static_cast<uint32_t>(__popcll(bal & ((1ull << lane) - 1)))] = S.buf[i];
        at += static_cast<uint32_t>(__popcll(bal));
    }
    if (tid == 0) a.uniq[b] = distinct;
}

// Longer segments, listed by class: a workgroup of 512 takes one of more than
// 512 values, or eight shorter ones, a wave each; one of 1,024 takes one of
// more than 4,096.  The grid is for n_med and n_mid (n_big) segments, which is
// more than there are when the host did not wait for the lists' lengths.
//
// Bound by LDS latency, so by the waves that fit a CU: 24 with 49 KB for eight
// waves and at most 80 registers.  On R-MAT graphs of 2^24 (2^27) vertices the
// segments of 513 to 4,096 values take 0.74 (6.6) ms, with 88 registers and 16
// waves 1.00 (9.4), by radix passes alone 1.49 (11.8).
__global__ void __launch_bounds__(kMedBlock, 6) k_seg_medium(SegArgs a, uint32_t n_med) {
    extern __shared__ uint64_t smem_med[];
    if (blockIdx.x < n_med) {
        if (blockIdx.x < *a.n_med) sort_segment<kMedBlock>(a, smem_med, a.l_med[blockIdx.x]);
        return;
    }
    const uint32_t wv = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6)));
    const uint32_t i = (blockIdx.x - n_med) * kMedWaves + wv;
    if (i < *a.n_mid) sort_segment<64>(a, smem_med + wv * (SegSmem<64>::bytes() / 8), a.l_mid[i]);
}

// The shorter class on its own, in 7 KB a wave (22 waves a CU): 0.21 (1.5) ms
// on the same graphs, by radix passes 0.48 (3.9).
__global__ void __launch_bounds__(64) k_seg_mid(SegArgs a) {
    extern __shared__ uint64_t smem_mid[];
    if (blockIdx.x < *a.n_mid) sort_segment<64>(a, smem_mid, a.l_mid[blockIdx.x]);
}

__global__ void __launch_bounds__(kBigBlock) k_seg_big(SegArgs a) {
    extern __shared__ uint64_t smem_big[];
    if (blockIdx.x < *a.n_big) sort_segment<kBigBlock>(a, smem_big, a.l_big[blockIdx.x]);
}

// ------------------------------------------------------------ set-up passes

// Every vertex with out-edges claims deg(v) values of its block's segment
// (a dead vertex has no edges: staging rejects such graphs).
__global__ void __launch_bounds__(kBlock) k_seg_claim(const uint32_t* __restrict__ row_off,
                                                      const uint32_t* __restrict__ bid, uint32_t n,
                                                      uint32_t* __restrict__ ecount, uint32_t* __restrict__ voff) {
    const uint32_t v = blockIdx.x * kBlock + threadIdx.x;
    if (v >= n) return;
    const uint32_t d = row_off[v + 1] - row_off[v];
    const uint32_t b = bid[v];
    if (d && b != 0xFFFFFFFFu) voff[v] = atomicAdd(&ecount[b], d);
}

struct FillShared {
    uint32_t base[kTileMaxVerts];
    alignas(8) uint8_t owner[kTileMaxEdges];
};

// Every edge (v, l, w) writes l << bb | block(w) into v's claimed range: one
// wave per tile, the eight gathers of a lane in flight together; longer rows
// by workgroups.
template <typename LabT>
__global__ void __launch_bounds__(kBlock) k_seg_fill(
    LongRows rows, const uint32_t* __restrict__ tgt, const LabT* __restrict__ lab,
    const uint32_t* __restrict__ bid, const uint32_t* __restrict__ bid_dst, const uint32_t* __restrict__ estart,
    const uint32_t* __restrict__ voff, const uint4* __restrict__ tiles, const uint32_t* __restrict__ act,
    const uint32_t* __restrict__ act_off, uint32_t n_tiles, int bb, uint64_t* __restrict__ vals) {
    __shared__ FillShared sh[kWaves];
    const uint32_t tid = threadIdx.x;
    if (blockIdx.x < rows.blocks()) {
        uint32_t e0, e1;
        const uint32_t v = rows.share(blockIdx.x, &e0, &e1);
        uint64_t* out = vals + estart[bid[v]] + voff[v] + (e0 - rows.row_off[v]);
        for (uint32_t e = e0 + tid; e < e1; e += kBlock)
            out[e - e0] = (static_cast<uint64_t>(lab[e]) << bb) | bid_dst[tgt[e]];
        return;
    }
    const uint32_t lane = lane_id();
    const uint32_t wv = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(tid >> 6)));
    const uint32_t tile = (blockIdx.x - rows.blocks()) * kWaves + wv;
    if (tile >= n_tiles) return;
    FillShared& S = sh[wv];
    const uint4 td = tiles[tile];
    const uint32_t nv = td.y - td.x, ne = td.w - td.z;
    uint32_t w[kLaneEdges], l[kLaneEdges];
#pragma unroll
    for (int q = 0; q < kLaneEdges; q++) {
        const uint32_t j = q * 64 + lane;
        w[q] = l[q] = 0;
        if (j < ne) {
            w[q] = __builtin_nontemporal_load(&tgt[td.z + j]);
            l[q] = static_cast<uint32_t>(__builtin_nontemporal_load(&lab[td.z + j]));
        }
    }
    uint32_t off = 0;
    if (lane < nv) {
        const uint32_t v = act[td.x + lane];
        off = act_off[td.x + lane] - td.z;
        // the value of local edge j of this vertex goes to base + j (mod 2^32)
        S.base[lane] = estart[bid[v]] + voff[v] - off;
    }
#pragma unroll
    for (int q = 0; q < kLaneEdges; q++) w[q] = q * 64 + lane < ne ? bid_dst[w[q]] : 0u;
    tile_owners(S.owner, lane < nv, off);
#pragma unroll
    for (int q = 0; q < kLaneEdges; q++) {
        const uint32_t j = q * 64 + lane;
        if (j < ne) vals[S.base[S.owner[j]] + j] = (static_cast<uint64_t>(l[q]) << bb) | w[q];
    }
}

// Size classes: single values are final; medium and large segments are
// listed (list order is free).  A workgroup takes kClassPerBlock segments and
// reserves its list entries with one atomic per class: an atomic per wave on
// one line of counters took 1.06 ms over 53 million segments, this takes
// 0.17 ms.
constexpr int kClassPerThread = 8;
constexpr uint32_t kClassPerBlock = kBlock * kClassPerThread;

__global__ void __launch_bounds__(kBlock) k_seg_class(const uint32_t* __restrict__ estart, uint32_t nb,
                                                      uint32_t* __restrict__ uniq, uint32_t* __restrict__ l_mid,
                                                      uint32_t* __restrict__ l_med, uint32_t* __restrict__ l_big,
                                                      uint32_t* __restrict__ l_huge, FinalHost* __restrict__ ctr) {
    __shared__ uint32_t s_n[4], s_at[4], s_huge;
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kClassPerBlock;
    if (threadIdx.x < 4) s_n[threadIdx.x] = 0;
    if (threadIdx.x == 4) s_huge = 0;
    __syncthreads();
    uint32_t cls[kClassPerThread], pos[kClassPerThread];
#pragma unroll
    for (int r = 0; r < kClassPerThread; r++) {
        const uint64_t b = base + r * kBlock + threadIdx.x;
        cls[r] = pos[r] = 0;
        if (b >= nb) continue;
        const uint32_t sz = estart[b + 1] - estart[b];
        if (sz <= 1) uniq[b] = sz;
        cls[r] = sz > kSegBigMax ? 4u : sz > kSegMedMax ? 3u : sz > kSegMidMax ? 2u : sz > kSegSmallMax ? 1u : 0u;
        if (cls[r]) pos[r] = atomicAdd(&s_n[cls[r] - 1], 1u);
        if (cls[r] == 4) atomicAdd(&s_huge, sz);
    }
    __syncthreads();
    if (threadIdx.x < 4 && s_n[threadIdx.x]) {
        uint32_t* c[4] = {ctr->mid, ctr->med, ctr->big, ctr->huge};
        s_at[threadIdx.x] = atomicAdd(c[threadIdx.x], s_n[threadIdx.x]);
    }
    if (threadIdx.x == 4 && s_huge) atomicAdd(ctr->huge_values, s_huge);
    __syncthreads();
    uint32_t* lists[4] = {l_mid, l_med, l_big, l_huge};
#pragma unroll
    for (int r = 0; r < kClassPerThread; r++)
        if (cls[r])
            lists[cls[r] - 1][s_at[cls[r] - 1] + pos[r]] = static_cast<uint32_t>(base + r * kBlock + threadIdx.x);
}

// tf[t] = first b in [0, nb] with off[b] >= t * T + c, for t < n_t (off is
// nondecreasing with nb + 1 entries and every searched point is <= off[nb]).
// Thread b writes the tiles whose point falls in (off[b - 1], off[b]].
__global__ void __launch_bounds__(kBlock) k_tile_first(const uint32_t* __restrict__ off, uint32_t nb, uint32_t T,
                                                       uint32_t c, uint32_t n_t, uint32_t* __restrict__ tf) {
    const uint32_t b = blockIdx.x * kBlock + threadIdx.x;
    if (b > nb) return;
    const int64_t lo_x = b == 0 ? 0 : static_cast<int64_t>(off[b - 1]) + 1;
    const int64_t hi_x = off[b];
    int64_t t0 = lo_x - static_cast<int64_t>(c);
    t0 = t0 <= 0 ? 0 : (t0 + T - 1) / T;
    const int64_t t1x = hi_x - static_cast<int64_t>(c);
    if (t1x < 0) return;
    const int64_t t1 = t1x / T < static_cast<int64_t>(n_t) - 1 ? t1x / T : static_cast<int64_t>(n_t) - 1;
    for (int64_t t = t0; t <= t1; t++) tf[t] = b;
}

// ------------------------------------------------------------ huge segments

__global__ void __launch_bounds__(kBlock) k_huge_sizes(const uint32_t* __restrict__ list, uint32_t nh,
                                                       const uint32_t* __restrict__ estart,
                                                       uint32_t* __restrict__ sz) {
    const uint32_t o = blockIdx.x * kBlock + threadIdx.x;
    if (o < nh) sz[o] = estart[list[o] + 1] - estart[list[o]];
}

// The keys of all huge segments, kHugeRun consecutive ones per workgroup, which
// lie in at most two segments.  Bound by the copy.  A workgroup per segment
// took as long as the longest one, 1.27 ms on an R-MAT graph of 2^27 vertices
// and 312 us on one of 2^24; this takes 263 and 23 us.
constexpr uint32_t kHugeRun = kBlock * 16;
static_assert(kHugeRun <= kSegBigMax, "a run meets at most two huge segments");

__global__ void __launch_bounds__(kBlock) k_huge_gather(const uint32_t* __restrict__ list, uint32_t nh,
                                                        const uint32_t* __restrict__ hstart, uint32_t m,
                                                        const uint32_t* __restrict__ estart,
                                                        const uint64_t* __restrict__ vals, int vb,
                                                        uint64_t* __restrict__ keys) {
    const uint64_t p0 = static_cast<uint64_t>(blockIdx.x) * kHugeRun;
    const uint32_t o0 = last_le(hstart, 0, nh, static_cast<uint32_t>(p0));
    const uint32_t next = o0 + 1 < nh ? hstart[o0 + 1] : m;
    const uint64_t* from0 = vals + (static_cast<int64_t>(estart[list[o0]]) - hstart[o0]);
    const uint64_t* from1 = next < m ? vals + (static_cast<int64_t>(estart[list[o0 + 1]]) - next) : from0;
    const uint64_t p1 = min(p0 + kHugeRun, static_cast<uint64_t>(m));
#pragma unroll 4
    for (uint64_t p = p0 + threadIdx.x; p < p1; p += kBlock) {
        const bool second = p >= next;
        keys[p] = static_cast<uint64_t>(o0 + (second ? 1u : 0u)) << vb | (second ? from1 : from0)[p];
    }
}

__global__ void __launch_bounds__(kBlock) k_huge_first(const uint64_t* __restrict__ keys, uint32_t m,
                                                       uint32_t* __restrict__ flag) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < m) flag[i] = (i == 0 || keys[i] != keys[i - 1]) ? 1u : 0u;
}

__global__ void __launch_bounds__(kBlock) k_huge_write(const uint64_t* __restrict__ keys, uint32_t m,
                                                       const uint32_t* __restrict__ flag,
                                                       const uint32_t* __restrict__ pos,
                                                       const uint32_t* __restrict__ list,
                                                       const uint32_t* __restrict__ hstart,
                                                       const uint32_t* __restrict__ estart, int vb,
                                                       uint64_t* __restrict__ vals) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= m || !flag[i]) return;
    const uint64_t k = keys[i];
    const uint32_t o = static_cast<uint32_t>(k >> vb);
    vals[estart[list[o]] + pos[i] - pos[hstart[o]]] = k & ((1ull << vb) - 1);
}

__global__ void __launch_bounds__(kBlock) k_huge_uniq(const uint32_t* __restrict__ list, uint32_t nh,
                                                      const uint32_t* __restrict__ hstart,
                                                      const uint32_t* __restrict__ pos,
                                                      const uint32_t* __restrict__ pos_total,
                                                      uint32_t* __restrict__ uniq) {
    const uint32_t o = blockIdx.x * kBlock + threadIdx.x;
    if (o >= nh) return;
    const uint32_t end = o + 1 < nh ? pos[hstart[o + 1]] : *pos_total;
    uniq[list[o]] = end - pos[hstart[o]];
}

// ------------------------------------------------------------ unpack

// Output positions [t U, (t + 1) U): the distinct values of block b occupy
// [ostart[b], ostart[b + 1]) and sit at the front of its segment.
__global__ void __launch_bounds__(kBlock) k_seg_unpack(const uint64_t* __restrict__ vals,
                                                       const uint32_t* __restrict__ estart,
                                                       const uint32_t* __restrict__ ostart, uint32_t nb,
                                                       const uint32_t* __restrict__ tile_first, uint32_t n_tiles,
                                                       uint32_t nse, int bb, uint32_t* __restrict__ s,
                                                       uint32_t* __restrict__ l, uint32_t* __restrict__ d) {
    __shared__ uint32_t s_off[kUnpackCache + 1];
    const uint32_t t = blockIdx.x;
    // blocks [b0, b1] hold the tile's outputs: b0 holds position t U
    const uint32_t b0 = tile_first[t] - 1;
    const uint32_t b1 = t + 1 < n_tiles ? tile_first[t + 1] - 1 : nb - 1;
    const uint32_t nbk = b1 - b0 + 1;
    const bool cached = nbk <= kUnpackCache;
    if (cached)
        for (uint32_t i = threadIdx.x; i <= nbk; i += kBlock) s_off[i] = ostart[b0 + i];
    __syncthreads();
    const uint64_t p0 = static_cast<uint64_t>(t) * kUnpackTile;
    const uint64_t p1 = min(p0 + kUnpackTile, static_cast<uint64_t>(nse));
    const uint32_t bmask = static_cast<uint32_t>((1ull << bb) - 1);
    for (uint64_t pp = p0 + threadIdx.x; pp < p1; pp += kBlock) {
        const uint32_t p = static_cast<uint32_t>(pp);
        const uint32_t b = cached ? b0 + last_le(s_off, 0, nbk, p) : last_le(ostart, b0, b1 + 1, p);
        const uint64_t v = vals[estart[b] + (p - ostart[b])];
        s[p] = b;
        l[p] = static_cast<uint32_t>(v >> bb);
        d[p] = static_cast<uint32_t>(v) & bmask;
    }
}

}  // namespace

bool bucketed_summary_edges_fit(const Staged& g, int lb, int bb) {
    const int vb = lb + bb;
    if (g.src || g.m == 0 || g.n_tiles + g.n_solo + g.n_hubs == 0) return false;
    // huge segments are ranked: at most m / (kSegBigMax + 1) of them
    return vb + bit_width(g.m / (kSegBigMax + 1)) <= 64;
}

void bucketed_summary_edges(const Staged& g, const uint32_t* bid, uint32_t nb, const uint32_t* dst_ids, int lb,
                            int bb, uint32_t* ecount, FinalOut& out, FinalHost* dev,
                            const std::function<const FinalHost&()>& fetch, Arena& arena, Arena& keep,
                            hipStream_t s) {
    const uint32_t n = g.n;
    const uint32_t m = static_cast<uint32_t>(g.m);
    const int vb = lb + bb;
    // 1. segments: per-vertex claims, then their placement (every edge
    // leaves an alive vertex, so the segments hold m values)
    uint32_t* voff = arena.alloc<uint32_t>(n);
    uint32_t* estart = arena.alloc<uint32_t>(static_cast<size_t>(nb) + 1);
    k_seg_claim<<<ceil_div(n, kBlock), kBlock, 0, s>>>(g.row_off, bid, n, ecount, voff);
    scan_exclusive(ecount, estart, nb, estart + nb, arena, s);
    // 2. values
    uint64_t* vals = arena.alloc<uint64_t>(m);
    const LongRows rows = long_rows(g);
    const uint32_t grid = rows.blocks() + ceil_div(g.n_tiles, kWaves);
    if (g.label_bytes == 2)
        k_seg_fill<uint16_t><<<grid, kBlock, 0, s>>>(rows, g.tgt, static_cast<const uint16_t*>(g.lab), bid, dst_ids,
                                                     estart, voff, g.tiles, g.act, g.act_off, g.n_tiles, bb, vals);
    else
        k_seg_fill<uint32_t><<<grid, kBlock, 0, s>>>(rows, g.tgt, static_cast<const uint32_t*>(g.lab), bid, dst_ids,
                                                     estart, voff, g.tiles, g.act, g.act_off, g.n_tiles, bb, vals);
    // 3. size classes
    uint32_t* uniq = arena.alloc<uint32_t>(static_cast<size_t>(nb) + 1);
    // at most this many segments hold more than `above` values
    auto list_cap = [&](uint32_t above) {
        return static_cast<uint32_t>(std::min<uint64_t>(nb, m / (above + 1ull)));
    };
    const uint32_t cap_mid = list_cap(kSegSmallMax), cap_med = list_cap(kSegMidMax), cap_big = list_cap(kSegMedMax),
                   cap_huge = list_cap(kSegBigMax);
    uint32_t* l_mid = arena.alloc<uint32_t>(cap_mid);
    uint32_t* l_med = arena.alloc<uint32_t>(cap_med);
    uint32_t* l_big = arena.alloc<uint32_t>(cap_big);
    uint32_t* l_huge = arena.alloc<uint32_t>(cap_huge);
    k_seg_class<<<ceil_div(nb, kClassPerBlock), kBlock, 0, s>>>(estart, nb, uniq, l_mid, l_med, l_big, l_huge,
                                                                dev);
    hip_check(hipGetLastError(), "segment launch");
    SegArgs a{};
    a.vals = vals;
    a.estart = estart;
    a.nb = nb;
    a.uniq = uniq;
    a.vb = vb;
    const uint32_t n_st = ceil_div(m, kSmallRange);
    {
        uint32_t* tf = arena.alloc<uint32_t>(n_st);
        k_tile_first<<<ceil_div(static_cast<uint64_t>(nb) + 1, kBlock), kBlock, 0, s>>>(estart, nb, kSmallRange, 0,
                                                                                       n_st, tf);
        a.tile_first = tf;
        a.n_tiles = n_st;
        k_seg_small<<<n_st, kSmallBlock, 0, s>>>(a);
    }
    // the lists' lengths, while the small segments are sorted; a graph too
    // small for a huge segment launches as many workgroups as its lists can
    // hold instead (at most 127, 31 and 3) and does not wait
    uint32_t n_mid = cap_mid, n_med = cap_med, n_big = cap_big, n_huge = 0, huge_elems = 0;
    if (cap_huge) {
        const FinalHost& c = fetch();
        n_mid = c.mid[0], n_med = c.med[0], n_big = c.big[0], n_huge = c.huge[0], huge_elems = c.huge_values[0];
    }
    a.l_mid = l_mid, a.l_med = l_med, a.l_big = l_big;
    a.n_mid = dev->mid, a.n_med = dev->med, a.n_big = dev->big;
    if (n_mid > kMidApart) {
        k_seg_mid<<<n_mid, 64, SegSmem<64>::bytes(), s>>>(a);
        n_mid = 0;
    }
    if (n_med || n_mid) {
        constexpr uint64_t with_mid = kMedWaves * SegSmem<64>::bytes();
        constexpr uint64_t med = SegSmem<kMedBlock>::bytes();
        static_assert(std::max(with_mid, med) <= 65536, "LDS without an attribute");
        k_seg_medium<<<n_med + ceil_div(n_mid, kMedWaves), kMedBlock, n_mid ? std::max(with_mid, med) : med, s>>>(a, n_med);
    }
    if (n_big) {
        const uint64_t bytes = SegSmem<kBigBlock>::bytes();
        hip_check(hipFuncSetAttribute(reinterpret_cast<const void*>(k_seg_big),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes)),
                  "large-segment LDS");
        k_seg_big<<<n_big, kBigBlock, bytes, s>>>(a);
    }
    hip_check(hipGetLastError(), "segment sort launch");
    if (n_huge) {
        uint32_t* hsz = arena.alloc<uint32_t>(static_cast<size_t>(n_huge) + 1);
        uint32_t* hstart = arena.alloc<uint32_t>(static_cast<size_t>(n_huge) + 1);
        k_huge_sizes<<<ceil_div(n_huge, kBlock), kBlock, 0, s>>>(l_huge, n_huge, estart, hsz);
        scan_exclusive(hsz, hstart, n_huge, hstart + n_huge, arena, s);
        uint64_t* ka = arena.alloc<uint64_t>(huge_elems);
        uint64_t* kb = arena.alloc<uint64_t>(huge_elems);
        k_huge_gather<<<ceil_div(huge_elems, kHugeRun), kBlock, 0, s>>>(l_huge, n_huge, hstart, huge_elems, estart, vals,
                                                                        vb, ka);
        uint64_t* sorted = radix_sort(ka, kb, huge_elems, bit_width(n_huge - 1) + vb, arena, s);
        // the other buffer holds the first-occurrence flags and their scan
        uint32_t* flag = reinterpret_cast<uint32_t*>(sorted == ka ? kb : ka);
        uint32_t* pos = flag + huge_elems;
        uint32_t* pos_total = arena.alloc<uint32_t>(1);
        const uint32_t gh = ceil_div(huge_elems, kBlock);
        k_huge_first<<<gh, kBlock, 0, s>>>(sorted, huge_elems, flag);
        scan_exclusive(flag, pos, huge_elems, pos_total, arena, s);
        k_huge_write<<<gh, kBlock, 0, s>>>(sorted, huge_elems, flag, pos, l_huge, hstart, estart, vb, vals);
        k_huge_uniq<<<ceil_div(n_huge, kBlock), kBlock, 0, s>>>(l_huge, n_huge, hstart, pos, pos_total, uniq);
        hip_check(hipGetLastError(), "huge segment launch");
    }
    // 4. output placement
    uint32_t* ostart = arena.alloc<uint32_t>(static_cast<size_t>(nb) + 1);
    scan_exclusive(uniq, ostart, nb, ostart + nb, arena, s, dev->edges);
    const FinalHost* c = &fetch();
    const uint32_t nse = c->edges[0];
    out.n_se = nse;
    if (!out.preset) {
        out.se_src = keep.alloc<uint32_t>(nse);
        out.se_label = keep.alloc<uint32_t>(nse);
        out.se_dst = keep.alloc<uint32_t>(nse);
    }
    const uint32_t n_ut = ceil_div(nse, kUnpackTile);
    if (n_ut) {
        uint32_t* tf = arena.alloc<uint32_t>(n_ut);
        k_tile_first<<<ceil_div(static_cast<uint64_t>(nb) + 1, kBlock), kBlock, 0, s>>>(ostart, nb, kUnpackTile, 1,
                                                                                       n_ut, tf);
        k_seg_unpack<<<n_ut, kBlock, 0, s>>>(vals, estart, ostart, nb, tf, n_ut, nse, bb, out.se_src, out.se_label,
                                             out.se_dst);
    }
    hip_check(hipGetLastError(), "unpack launch");
}

}  // namespace bsim

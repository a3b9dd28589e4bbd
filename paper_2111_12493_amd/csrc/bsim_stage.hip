// bsim_stage.hip -- staging of a graph for the refinement kernels (a1) and
// the device prefix sum the library uses.
//
// Staging validates the CSR (paper Sec. 3.1 Phase 0 co-locates every vertex
// with its out-edges; here that is the out-edge CSR itself) and cuts the vertex
// range into tiles, solo vertices and hub buckets:
//   * a vertex of 1..kTileMaxEdges out-edges belongs to exactly one tile, a
//     run of consecutive such vertices packed greedily (within kStageVerts
//     vertices) up to kTileMaxEdges edges and kTileMaxVerts vertices;
//   * one of up to kSoloMaxEdges is a workgroup's work by itself;
//   * one of more is a hub: of degree d it is cut into chunks of kChunkEdges
//     edges that write its mixed pair keys to d scratch slots, and into 2^b
//     hash buckets that each fit the LDS table of the hub-bucket launch.
#include <algorithm>

#include "bsim_resolve.h"  // host_radix_sort
#include "bsim_device.h"

namespace bsim {

// ------------------------------------------------------------------ scan

namespace {

constexpr int kScanItems = 4;
constexpr int kScanTile = kBlock * kScanItems;  // 1024 values per block

__device__ inline uint32_t wave_incl_scan(uint32_t x) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// Exclusive scan of one value per thread across the block; returns the
// thread's exclusive prefix and the block total in *total.
__device__ inline uint32_t block_excl_scan(uint32_t x, uint32_t* total) {
    __shared__ uint32_t s_w[kBlock / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t inc = wave_incl_scan(x);
    if (lane == 63) s_w[wid] = inc;
    __syncthreads();
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kBlock / 64; i++) {
        if (i < wid) off += s_w[i];
        tot += s_w[i];
    }
    __syncthreads();
    *total = tot;
    return off + inc - x;
}

__global__ void __launch_bounds__(kBlock) k_scan_reduce(const uint32_t* __restrict__ in, uint32_t n,
                                                        uint32_t* __restrict__ sums) {
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kScanTile;
    uint32_t x = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; i++) {
        uint64_t j = base + static_cast<uint64_t>(i) * kBlock + threadIdx.x;
        if (j < n) x += in[j];
    }
    uint32_t tot;
    (void)block_excl_scan(x, &tot);
    if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// Up to kScanSmall values in one launch of one workgroup: three launches take
// some 15 us in a stream of small kernels whatever they do, this one 4 to 6.
constexpr uint32_t kScanSmallItems = 16;
constexpr uint32_t kScanSmall = 1024 * kScanSmallItems;

__global__ void __launch_bounds__(1024) k_scan_small(const uint32_t* in, uint32_t* out, uint32_t n,
                                                     uint32_t* total, uint32_t* total2) {
    __shared__ uint32_t s_w[16];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const uint32_t per = (n + 1023) / 1024;  // <= kScanSmallItems
    const uint32_t j0 = tid * per;
    uint32_t v[kScanSmallItems], x = 0;
#pragma unroll
    for (uint32_t i = 0; i < kScanSmallItems; i++) {
        v[i] = i < per && j0 + i < n ? in[j0 + i] : 0u;
        x += v[i];
    }
    const uint32_t inc = wave_incl_scan(x);
    if (lane == 63) s_w[wid] = inc;
    __syncthreads();
    uint32_t run = inc - x, tot = 0;
    for (uint32_t i = 0; i < 16; i++) {
        if (i < wid) run += s_w[i];
        tot += s_w[i];
    }
#pragma unroll
    for (uint32_t i = 0; i < kScanSmallItems; i++) {
        if (i < per && j0 + i < n) out[j0 + i] = run;
        run += v[i];
    }
    if (tid == 0 && total) *total = tot;
    if (tid == 0 && total2) *total2 = tot;
}

__global__ void __launch_bounds__(1024) k_scan_spine(uint32_t* __restrict__ sums, uint32_t nb,
                                                    uint32_t* __restrict__ total, uint32_t* __restrict__ total2) {
    __shared__ uint32_t s_w[16];
    __shared__ uint32_t s_carry;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (threadIdx.x == 0) s_carry = 0;
    __syncthreads();
    for (uint32_t base = 0; base < nb; base += 1024) {
        uint32_t j = base + threadIdx.x;
        uint32_t x = j < nb ? sums[j] : 0;
        uint32_t inc = wave_incl_scan(x);
        if (lane == 63) s_w[wid] = inc;
        __syncthreads();
        uint32_t off = 0, tot = 0;
        for (int i = 0; i < 16; i++) {
            if (i < wid) off += s_w[i];
            tot += s_w[i];
        }
        uint32_t carry = s_carry;
        if (j < nb) sums[j] = carry + off + inc - x;
        __syncthreads();
        if (threadIdx.x == 0) s_carry = carry + tot;
        __syncthreads();
    }
    if (threadIdx.x == 0 && total) *total = s_carry;
    if (threadIdx.x == 0 && total2) *total2 = s_carry;
}

__global__ void __launch_bounds__(kBlock) k_scan_down(const uint32_t* in, uint32_t* out, uint32_t n,
                                                      const uint32_t* __restrict__ sums) {
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * kScanTile +
                          static_cast<uint64_t>(threadIdx.x) * kScanItems;
    uint32_t v[kScanItems];
    uint32_t x = 0;
#pragma unroll
    for (int i = 0; i < kScanItems; i++) {
        v[i] = (base + i < n) ? in[base + i] : 0;
        x += v[i];
    }
    uint32_t tot;
    uint32_t run = block_excl_scan(x, &tot) + sums[blockIdx.x];
#pragma unroll
    for (int i = 0; i < kScanItems; i++) {
        if (base + i < n) out[base + i] = run;
        run += v[i];
    }
}

}  // namespace

void scan_exclusive(const uint32_t* in, uint32_t* out, uint32_t n, uint32_t* total_dev,
                    Arena& arena, hipStream_t s, uint32_t* total2_dev) {
    if (n <= kScanSmall) {
        k_scan_small<<<1, 1024, 0, s>>>(in, out, n, total_dev, total2_dev);
        hip_check(hipGetLastError(), "scan launch");
        return;
    }
    uint32_t nb = ceil_div(n, kScanTile);
    uint32_t* sums = arena.alloc<uint32_t>(nb);
    k_scan_reduce<<<nb, kBlock, 0, s>>>(in, n, sums);
    k_scan_spine<<<1, 1024, 0, s>>>(sums, nb, total_dev, total2_dev);
    k_scan_down<<<nb, kBlock, 0, s>>>(in, out, n, sums);
    hip_check(hipGetLastError(), "scan launch");
}

// --------------------------------------------------------------- staging

namespace {

// Staging is two passes over the row offsets with a one-block scan between
// them, and one pass over the edges beside the first.  A workgroup owns
// kStageVerts consecutive vertices: it classifies them (hub, solo, tile
// vertex, no out-edges), compacts the tile vertices' edge ranges in LDS and
// packs them into tiles, so a tile never leaves its workgroup's vertices.
// The first pass counts (hubs, tile vertices, solo vertices, tiles), the scan
// places the counts, the second pass repeats the work and writes the lists.
// Repeating it costs 4 bytes per vertex; carrying flags, positions and three
// separate scans and compactions between passes cost 72.
//
// Packing is greedy.  Row ends grow with the vertex, so the vertices that
// still fit a tile starting at edge a are a prefix (row end - a at most
// kTileMaxEdges; a solo vertex or hub between two tile vertices exceeds that
// by itself): one ballot of a wave finds a tile's end.  A
// single lane walking its window vertex by vertex took 106-185 us whatever
// the graph's size, twice per call.
//
// Bound: the row and type offsets once and the row offsets again, the lists
// written, and the edges once.  On 10,000 vertices and 50,000 edges the three
// kernels take 26 us where 19 launches took 410 us; on 2^27 vertices and
// 2^30 edges of 16-bit labels 3.3 ms (counting 2.10, scan 0.11, writing 1.09)
// where they took 7.1 ms.
constexpr uint32_t kStageVerts = 2048;
constexpr uint32_t kStageRounds = kStageVerts / kBlock;
constexpr uint32_t kStageGroups = kStageVerts / 64;  // 64-vertex groups: (round, wave)
static_assert(kStageGroups <= 64, "one wave scans the group counts");
static_assert(kTileMaxVerts == 64, "packing tests one ballot");

struct StageShared {
    uint32_t off[kStageVerts + 1];
    uint32_t a[kStageVerts];        // edge ranges of the tile vertices
    uint32_t b[kStageVerts];
    uint32_t act[kStageGroups];     // tile vertices, solo vertices and hubs per group
    uint32_t solo[kStageGroups];
    uint32_t hub[kStageGroups];
    uint32_t red[2 * kWaves];
};

struct StageArgs {
    const uint32_t* row_off;
    const uint32_t* type_off;
    const uint8_t* alive;
    uint32_t n;
    uint64_t m;
    const uint32_t* tgt;
    const void* lab;
    uint32_t n_vblk;     // vertex blocks (the grid's first)
    uint4* cnt;          // per vertex block: hubs, tile vertices, solo vertices, tiles
    uint4* seen;         // per block: error bits, most types, largest label
    uint32_t wide;       // tgt and lab are aligned for four edges per load
    uint32_t* act;
    uint32_t* act_off;
    uint32_t* iso;
    uint32_t* solo;
    uint32_t* hubs;      // (vertex, degree, first edge) each
    uint4* tiles;
    uint32_t hub_cap, solo_cap, tile_cap;
    RunStatus* status;
};

// Greedy packing of the na compacted edge ranges by one wave; returns the
// tile count.  out (nullable) receives positions base + i.
__device__ uint32_t pack_tiles(const StageShared& S, uint32_t na, uint32_t base, uint4* out, uint32_t room) {
    const uint32_t lane = threadIdx.x & 63;
    uint32_t made = 0;
    for (uint32_t start = 0; start < na; made++) {
        const uint32_t a0 = S.a[start];
        const uint32_t j = start + lane;
        const bool fits = j < na && S.b[j] - a0 <= static_cast<uint32_t>(kTileMaxEdges);
        uint32_t end = start + static_cast<uint32_t>(__popcll(__ballot(fits)));
        if (end == start) end = start + 1;  // offsets that are not monotone: the call fails later
        if (out && lane == 0 && made < room) out[made] = make_uint4(base + start, base + end, a0, S.b[end - 1]);
        start = end;
    }
    return made;
}

template <bool kEmit>
__device__ void stage_vertices(const StageArgs& a, StageShared& S) {
    const uint32_t tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const uint32_t base = blockIdx.x * kStageVerts;
    const uint32_t cnt = min(kStageVerts, a.n - base);
    for (uint32_t i = tid; i <= cnt; i += kBlock) S.off[i] = a.row_off[base + i];
    __syncthreads();
    uint32_t err = 0, types = 0, is_act = 0, is_solo = 0, is_hub = 0;  // bit r: round r's vertex
#pragma unroll
    for (uint32_t r = 0; r < kStageRounds; r++) {
        const uint32_t i = r * kBlock + tid, v = base + i;
        const bool in = i < cnt;
        uint32_t x = 0, y = 0;
        if (in) {
            x = S.off[i];
            y = S.off[i + 1];
            if (!kEmit) {
                const uint32_t t0 = a.type_off[v], t1 = a.type_off[v + 1];
                if (y < x || t1 < t0) err |= kErrInvalid;
                if (v == 0 && (x != 0 || t0 != 0)) err |= kErrInvalid;
                if (v == a.n - 1 && static_cast<uint64_t>(y) != a.m) err |= kErrInvalid;
                if (a.alive && y != x && !a.alive[v]) err |= kErrInvalid;
                types = max(types, t1 - t0);
            }
        }
        const uint32_t d = in && y > x ? y - x : 0u;
        const bool act = d && d <= static_cast<uint32_t>(kTileMaxEdges);
        const bool hub = d > kSoloMaxEdges, solo = d && !act && !hub;
        is_act |= static_cast<uint32_t>(act) << r;
        is_solo |= static_cast<uint32_t>(solo) << r;
        is_hub |= static_cast<uint32_t>(hub) << r;
        const uint64_t ba = __ballot(act), bs = __ballot(solo), bh = __ballot(hub);
        if (lane == 0) {
            S.act[r * kWaves + wv] = static_cast<uint32_t>(__popcll(ba));
            S.solo[r * kWaves + wv] = static_cast<uint32_t>(__popcll(bs));
            S.hub[r * kWaves + wv] = static_cast<uint32_t>(__popcll(bh));
        }
    }
    __syncthreads();
    // exclusive prefixes of the group counts, one group per lane
    const bool grp_lane = lane < kStageGroups;
    const uint32_t ca = grp_lane ? S.act[lane] : 0, cs = grp_lane ? S.solo[lane] : 0, ch = grp_lane ? S.hub[lane] : 0;
    const uint32_t ia = wave_incl_scan(ca), is = wave_incl_scan(cs), ih = wave_incl_scan(ch);
    auto from = [](uint32_t x, uint32_t l) {
        return static_cast<uint32_t>(__shfl(static_cast<int>(x), static_cast<int>(l), 64));
    };
    const uint32_t na = from(ia, 63), ns = from(is, 63), nh = from(ih, 63);
    uint4 at = make_uint4(0, 0, 0, 0);
    if (kEmit) at = a.cnt[blockIdx.x];
    const uint32_t iso_at = base - at.x - at.y - at.z;
#pragma unroll
    for (uint32_t r = 0; r < kStageRounds; r++) {
        const uint32_t i = r * kBlock + tid, v = base + i;
        const uint32_t grp = r * kWaves + wv;
        const bool act = (is_act >> r) & 1, solo = (is_solo >> r) & 1, hub = (is_hub >> r) & 1;
        const uint64_t lt = (1ull << lane) - 1;
        const uint32_t pa = from(ia - ca, grp) + static_cast<uint32_t>(__popcll(__ballot(act) & lt));
        if (act) {
            S.a[pa] = S.off[i];
            S.b[pa] = S.off[i + 1];
        }
        if (kEmit) {
            const uint32_t ps = from(is - cs, grp) + static_cast<uint32_t>(__popcll(__ballot(solo) & lt));
            const uint32_t ph = from(ih - ch, grp) + static_cast<uint32_t>(__popcll(__ballot(hub) & lt));
            if (act) {
                a.act[at.y + pa] = v;
                a.act_off[at.y + pa] = S.off[i];
            } else if (solo) {
                if (at.z + ps < a.solo_cap) a.solo[at.z + ps] = v;
            } else if (hub) {
                if (at.x + ph < a.hub_cap) {
                    uint32_t* h = a.hubs + 3ull * (at.x + ph);
                    h[0] = v;
                    h[1] = S.off[i + 1] - S.off[i];
                    h[2] = S.off[i];
                }
            } else if (i < cnt) {
                a.iso[iso_at + (i - pa - ps - ph)] = v;
            }
        }
    }
    if (!kEmit) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            types = max(types, static_cast<uint32_t>(__shfl_xor(static_cast<int>(types), d, 64)));
            err |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(err), d, 64));
        }
        if (lane == 0) S.red[wv] = err << 16 | min(types, 0xFFFFu);  // (more than 4,096 types are refused)
    }
    __syncthreads();
    if (wv == 0) {
        uint4* out = kEmit && at.w < a.tile_cap ? a.tiles + at.w : nullptr;
        const uint32_t made = pack_tiles(S, na, at.y, out, kEmit ? a.tile_cap - at.w : 0u);
        if (!kEmit && lane == 0) {
            a.cnt[blockIdx.x] = make_uint4(nh, na, ns, made);
            uint32_t e = 0, t = 0;
            for (int i = 0; i < kWaves; i++) {
                e |= S.red[i] >> 16;
                t = max(t, S.red[i] & 0xFFFFu);
            }
            a.seen[blockIdx.x] = make_uint4(e, t, 0, 0);
        }
    }
}

// Target range, deadness and the largest label over the edges of one block.
template <typename LabT>
__device__ void stage_edges(const StageArgs& a, uint32_t* s_red) {
    const LabT* __restrict__ lab = static_cast<const LabT*>(a.lab);
    const uint64_t tid0 = static_cast<uint64_t>(blockIdx.x - a.n_vblk) * kBlock + threadIdx.x;
    const uint64_t step = static_cast<uint64_t>(gridDim.x - a.n_vblk) * kBlock;
    uint32_t err = 0, mx = 0;
    auto edge = [&](uint32_t w, uint32_t l) {
        if (w >= a.n)
            err |= kErrRange;
        else if (a.alive && !a.alive[w])
            err |= kErrInvalid;
        mx = max(mx, l);
    };
    uint64_t done = 0;
    if (a.wide) {
        // four edges per load where both arrays allow it: the counting pass
        // over 2^27 vertices and 2^30 edges moves its 7.5 GB at 3.6 TB/s
        // (2.1 ms; with one edge per load, in two launches, 2.77 ms)
        struct alignas(4 * sizeof(LabT)) Lab4 {
            LabT x[4];
        };
        const uint4* t4 = reinterpret_cast<const uint4*>(a.tgt);
        const Lab4* l4 = reinterpret_cast<const Lab4*>(lab);
        for (uint64_t q = tid0; q < a.m / 4; q += step) {
            const uint4 w = t4[q];
            const Lab4 l = l4[q];
            edge(w.x, l.x[0]);
            edge(w.y, l.x[1]);
            edge(w.z, l.x[2]);
            edge(w.w, l.x[3]);
        }
        done = a.m / 4 * 4;
    }
    for (uint64_t e = done + tid0; e < a.m; e += step) edge(a.tgt[e], static_cast<uint32_t>(lab[e]));
    // reduce over the block before touching global memory
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        mx = max(mx, static_cast<uint32_t>(__shfl_xor(static_cast<int>(mx), d, 64)));
        err |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(err), d, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        s_red[threadIdx.x >> 6] = mx;
        s_red[kWaves + (threadIdx.x >> 6)] = err;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kWaves; i++) {
            mx = max(mx, s_red[i]);
            err |= s_red[kWaves + i];
        }
        a.seen[blockIdx.x] = make_uint4(err, 0, mx, 0);
    }
}

template <typename LabT>
__global__ void __launch_bounds__(kBlock) k_stage_count(StageArgs a) {
    __shared__ StageShared S;
    if (blockIdx.x < a.n_vblk)
        stage_vertices<false>(a, S);
    else
        stage_edges<LabT>(a, S.red);
}

__global__ void __launch_bounds__(kBlock) k_stage_emit(StageArgs a) {
    __shared__ StageShared S;
    // malformed offsets: the counts mean nothing, and the call fails
    if (a.status->error & kErrInvalid) return;
    stage_vertices<true>(a, S);
}

// Exclusive scan of the per-block counts in place, totals to total[0..3]; and
// the status from what the nseen blocks saw.
constexpr uint32_t kSpineItems = 4;

__global__ void __launch_bounds__(1024) k_stage_spine(uint4* cnt, uint32_t nb, const uint4* __restrict__ seen,
                                                      uint32_t nseen, RunStatus* status, uint32_t* total) {
    __shared__ uint4 s_w[16];
    const uint32_t lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint4 carry = make_uint4(0, 0, 0, 0);
    auto add = [](uint4 x, uint4 y) { return make_uint4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w); };
    for (uint64_t b0 = 0; b0 < nb; b0 += 1024 * kSpineItems) {
        const uint64_t j0 = b0 + static_cast<uint64_t>(threadIdx.x) * kSpineItems;
        uint4 v[kSpineItems], sum = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (uint32_t i = 0; i < kSpineItems; i++) {
            v[i] = j0 + i < nb ? cnt[j0 + i] : make_uint4(0, 0, 0, 0);
            sum = add(sum, v[i]);
        }
        const uint4 inc = make_uint4(wave_incl_scan(sum.x), wave_incl_scan(sum.y), wave_incl_scan(sum.z),
                                     wave_incl_scan(sum.w));
        if (lane == 63) s_w[wid] = inc;
        __syncthreads();
        uint4 run = carry;
        for (uint32_t i = 0; i < 16; i++) {
            const uint4 t = s_w[i];
            if (i < wid) run = add(run, t);
            carry = add(carry, t);
        }
        run = make_uint4(run.x + inc.x - sum.x, run.y + inc.y - sum.y, run.z + inc.z - sum.z,
                         run.w + inc.w - sum.w);
#pragma unroll
        for (uint32_t i = 0; i < kSpineItems; i++) {
            if (j0 + i < nb) cnt[j0 + i] = run;
            run = add(run, v[i]);
        }
        __syncthreads();
    }
    uint32_t err = 0, types = 0, label = 0;
    for (uint32_t j = threadIdx.x; j < nseen; j += 1024) {
        const uint4 x = seen[j];
        err |= x.x;
        types = max(types, x.y);
        label = max(label, x.z);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        err |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(err), d, 64));
        types = max(types, static_cast<uint32_t>(__shfl_xor(static_cast<int>(types), d, 64)));
        label = max(label, static_cast<uint32_t>(__shfl_xor(static_cast<int>(label), d, 64)));
    }
    if (lane == 0) s_w[wid] = make_uint4(err, types, label, 0);
    __syncthreads();
    if (threadIdx.x == 0) {
        for (uint32_t i = 1; i < 16; i++) {
            err |= s_w[i].x;
            types = max(types, s_w[i].y);
            label = max(label, s_w[i].z);
        }
        *status = RunStatus{0, 0, 0, err, label, types, {0, 0}};
        total[0] = carry.x;
        total[1] = carry.y;
        total[2] = carry.z;
        total[3] = carry.w;
    }
}

__global__ void __launch_bounds__(kBlock) k_salt(uint64_t* salt, uint32_t count, uint32_t in_base) {
    const uint32_t l = blockIdx.x * kBlock + threadIdx.x;
    if (l < count) salt[l] = label_salt(l, in_base);
}

// The hub schedule, on the host (a graph of 2^30 edges has some 10^5 hubs):
// hubs by degree, largest first, so that long buckets start early.  info
// holds (vertex, degree, first edge) per hub in vertex order.
void schedule_hubs(Staged& g, const uint32_t* info, Arena& arena, hipStream_t s) {
    const uint32_t nh = g.n_hubs;
    // ties in hub order: a stable radix sort on the complemented degree (a
    // comparison sort takes milliseconds here)
    std::vector<uint32_t> order(nh);
    {
        std::vector<uint64_t> key(nh), k2;
        std::vector<uint32_t> v2;
        for (uint32_t i = 0; i < nh; i++) {
            key[i] = 0xFFFFFFFFull - info[3ull * i + 1];
            order[i] = i;
        }
        host_radix_sort(key, order, 32, k2, v2);
    }
    // a hub of degree d: ceil(d / kChunkEdges) chunk blocks, and 2^b bucket
    // blocks so that a bucket expects at most 11/12 of the keys that its
    // rounds take (2,816 of 3,072 by default, five standard deviations)
    const uint64_t per_bucket = std::max<uint64_t>(1, uint64_t(g.hub_table_slots) * 11 / 16);
    uint32_t n_chunks = 0, n_blocks = 0;
    std::vector<uint32_t> logb(nh, 0);
    for (uint32_t i = 0; i < nh; i++) {
        const uint32_t d = info[3ull * order[i] + 1];
        const uint64_t want = (d + per_bucket - 1) / per_bucket;
        logb[i] = std::min<uint32_t>(static_cast<uint32_t>(bit_width(next_pow2(want)) - 1), kMaxHubLogB);
        n_chunks += ceil_div(d, kChunkEdges);
        n_blocks += 1u << logb[i];
    }
    // every array of the schedule in one upload
    std::vector<uint32_t> up(6ull * nh + 2ull * n_chunks + 2ull * n_blocks);
    uint64_t* key_off = reinterpret_cast<uint64_t*>(up.data());  // first: 8-byte entries
    uint32_t* hv = up.data() + 2ull * nh;
    uint32_t *hl = hv + nh, *hc0 = hl + nh, *hnc = hc0 + nh;
    uint32_t *ch = hnc + nh, *ce = ch + n_chunks, *bh = ce + n_chunks, *bb = bh + n_blocks;
    uint64_t keys = 0;
    uint32_t nc = 0, nb = 0;
    for (uint32_t i = 0; i < nh; i++) {
        const uint32_t* h = info + 3ull * order[i];
        hv[i] = h[0];
        hl[i] = logb[i];
        key_off[i] = keys;
        hc0[i] = nc;
        hnc[i] = ceil_div(h[1], kChunkEdges);
        keys += h[1];
        for (uint32_t c = 0; c < hnc[i]; c++) {
            ch[nc] = i;
            ce[nc++] = h[2] + c * kChunkEdges;
        }
        for (uint32_t b = 0; b < (1u << logb[i]); b++) {
            bh[nb] = i;
            bb[nb++] = b;
        }
    }
    uint32_t* d = arena.alloc<uint32_t>(up.size());
    // (pageable memory: the call returns once the source has been read)
    hip_check(hipMemcpyAsync(d, up.data(), up.size() * 4, hipMemcpyHostToDevice, s), "hub schedule");
    auto dev = [&](const uint32_t* host) { return d + (host - up.data()); };
    g.n_hub_chunks = n_chunks;
    g.n_hub_blocks = n_blocks;
    g.hub_keys_total = keys;
    g.hub_key_off = reinterpret_cast<uint64_t*>(d);
    g.hub_v = dev(hv);
    g.hub_logb = dev(hl);
    g.hub_chunk0 = dev(hc0);
    g.hub_nchunks = dev(hnc);
    g.hc_hub = dev(ch);
    g.hc_e0 = dev(ce);
    g.hb_hub = dev(bh);
    g.hb_bucket = dev(bb);
}

}  // namespace

void stage_graph(Staged& g, StageHost* host, Arena& arena, hipStream_t s) {
    const uint32_t n = g.n;
    // status, counts and hub list lie together, as in StageHost
    const uint32_t hub_cap = static_cast<uint32_t>(g.m / (kSoloMaxEdges + 1)) + 1;
    const uint32_t solo_cap = static_cast<uint32_t>(g.m / (kTileMaxEdges + 1)) + 1;
    const size_t head = sizeof(RunStatus) + sizeof(host->counts);
    uint8_t* dev = arena.alloc<uint8_t>(head + 12ull * hub_cap);
    RunStatus* status = reinterpret_cast<RunStatus*>(dev);
    uint32_t* counts = reinterpret_cast<uint32_t*>(dev + sizeof(RunStatus));
    uint32_t* hubs = reinterpret_cast<uint32_t*>(dev + head);
    // tiles: one that its edges end is followed by a vertex with which it
    // would pass kTileMaxEdges (a vertex counts for its own tile and, first
    // in it, for the one before), one that its vertices end holds
    // kTileMaxVerts, one that a solo vertex or hub ends precedes that
    // vertex, and every workgroup's last tile may be short
    const uint32_t n_vblk = ceil_div(n, kStageVerts);
    const uint64_t tile_cap = 2 * g.m / (kTileMaxEdges + 1) + n / kTileMaxVerts + solo_cap + n_vblk + 1;
    StageArgs a{};
    a.row_off = g.row_off;
    a.type_off = g.type_off;
    a.alive = g.alive;
    a.n = n;
    a.m = g.m;
    a.tgt = g.tgt;
    a.lab = g.lab;
    a.n_vblk = n_vblk;
    const uint32_t n_eblk =
        n && g.m && !g.trusted ? std::min<uint32_t>(ceil_div(g.m, 4 * kBlock), 2048) : 0u;
    a.cnt = arena.alloc<uint4>(n_vblk + 1ull);
    a.seen = arena.alloc<uint4>(n_vblk + n_eblk + 1ull);
    a.wide = (reinterpret_cast<uintptr_t>(g.tgt) % 16 == 0 &&
              reinterpret_cast<uintptr_t>(g.lab) % (4 * g.label_bytes) == 0)
                 ? 1u
                 : 0u;
    a.act = g.act = arena.alloc<uint32_t>(n + 1ull);
    a.act_off = g.act_off = arena.alloc<uint32_t>(n + 1ull);
    a.iso = g.iso = arena.alloc<uint32_t>(n + 1ull);
    a.solo = g.solo_v = arena.alloc<uint32_t>(solo_cap);
    a.hubs = hubs;
    a.tiles = g.tiles = arena.alloc<uint4>(tile_cap);
    a.hub_cap = hub_cap;
    a.solo_cap = solo_cap;
    a.tile_cap = static_cast<uint32_t>(tile_cap);
    a.status = status;
    if (n > 0) {
        if (g.label_bytes == 2)
            k_stage_count<uint16_t><<<n_vblk + n_eblk, kBlock, 0, s>>>(a);
        else
            k_stage_count<uint32_t><<<n_vblk + n_eblk, kBlock, 0, s>>>(a);
    }
    k_stage_spine<<<1, 1024, 0, s>>>(a.cnt, n_vblk, a.seen, n_vblk + n_eblk, status, counts);
    if (n > 0) k_stage_emit<<<n_vblk, kBlock, 0, s>>>(a);
    hip_check(hipGetLastError(), "stage launch");
    // one copy brings the counts and, for most graphs, every hub
    const uint32_t with = std::min(hub_cap, kStageHubs);
    hip_check(hipMemcpyAsync(host, dev, head + 12ull * with, hipMemcpyDeviceToHost, s), "stage counts");
    hip_check(hipStreamSynchronize(s), "stage sync");
    if (host->st.error & kErrRange)
        throw DeviceError{BSIM_E_RANGE, "edge target out of range"};
    if (host->st.error & kErrInvalid)
        throw DeviceError{BSIM_E_INVALID, "malformed CSR or an edge touching a dead vertex"};
    if (host->st.max_types > 4096)
        throw DeviceError{BSIM_E_UNSUPPORTED, "more than 4096 type ids on one vertex"};
    if (host->st.max_label >= (1u << 24))
        throw DeviceError{BSIM_E_UNSUPPORTED, "edge labels must be < 2^24"};
    if (!g.trusted) g.max_label = host->st.max_label;
    g.n_hubs = host->counts[0];
    g.n_act = host->counts[1];
    g.n_solo = host->counts[2];
    g.n_tiles = host->counts[3];
    g.n_iso = n - g.n_hubs - g.n_act - g.n_solo;
    if (g.n_hubs > hub_cap || g.n_solo > solo_cap || g.n_tiles > tile_cap)
        throw DeviceError{BSIM_E_DEVICE, "internal: a staging list outgrew its bound"};
    g.n_hub_chunks = g.n_hub_blocks = 0;
    g.hub_keys_total = 0;
    if (g.n_hubs > with) {
        std::vector<uint32_t> all(3ull * g.n_hubs);
        hip_check(hipMemcpyAsync(all.data(), hubs, all.size() * 4, hipMemcpyDeviceToHost, s), "hubs");
        hip_check(hipStreamSynchronize(s), "hubs sync");
        schedule_hubs(g, all.data(), arena, s);
    } else if (g.n_hubs) {
        schedule_hubs(g, host->hubs, arena, s);
    }

    g.salt = arena.alloc<uint64_t>(g.max_label + 1ull);
}

void launch_salts(const Staged& g, hipStream_t s) {
    const uint32_t nsalt = g.max_label + 1;
    k_salt<<<ceil_div(nsalt, kBlock), kBlock, 0, s>>>(g.salt, nsalt, g.in_label_base);
    hip_check(hipGetLastError(), "salt launch");
}

}  // namespace bsim

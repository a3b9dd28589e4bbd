// Direction and label parameterizations (Sec. 2.4; backward bisimulation,
// Sec. 2.5) as graph views in front of the unchanged refinement kernels.
//
// From a staged, validated graph g the device builds
//   f  the kept edges: those whose label is in the label set P_l (g itself
//      when there is none), in their own direction; the summary edges are
//      taken from f;
//   h  the graph the signatures read: f itself (forward), f reversed
//      (backward: the pairs of w are its incoming edges (v, l, w)), or f
//      plus f reversed (both), the reversed copies on labels L + l with
//      L = max label + 1.  The salt table of h maps label L + l to
//      M(C_L + 2^31 + l), so an incoming l-edge is salted as an outgoing
//      edge of label l + 2^31 (a range input labels never reach).
// The reversal is a radix sort of the edges by target.  Counting the targets
// and scattering by a cursor per target, two atomics per edge, serializes on
// the hubs' counters: on R-MAT 2^22 / 2^25 that took 7.0 ms where the sort
// and its passes take 1.4.  The order of the edges within a row of h does
// not matter, since a signature is a set.
#include "bsim_device.h"

namespace bsim {
namespace {

__global__ void __launch_bounds__(kBlock) k_label_mask(const uint32_t* __restrict__ ids, uint32_t n_ids,
                                                       uint8_t* __restrict__ mask, uint32_t mask_size) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n_ids && ids[i] < mask_size) mask[ids[i]] = 1;
}

template <typename LabT>
__global__ void __launch_bounds__(kBlock) k_keep_flags(const LabT* __restrict__ lab, uint32_t m,
                                                       const uint8_t* __restrict__ mask,
                                                       uint32_t* __restrict__ keep) {
    const uint32_t e = blockIdx.x * kBlock + threadIdx.x;
    if (e < m) keep[e] = mask[static_cast<uint32_t>(lab[e])];
}

// Row offsets of the kept edges: f_row_off[v] = kept edges before row v.
__global__ void __launch_bounds__(kBlock) k_kept_rows(const uint32_t* __restrict__ row_off, uint32_t n, uint32_t m,
                                                      const uint32_t* __restrict__ kpos,
                                                      const uint32_t* __restrict__ m_kept,
                                                      uint32_t* __restrict__ f_row_off) {
    const uint32_t v = blockIdx.x * kBlock + threadIdx.x;
    if (v > n) return;
    const uint32_t e = row_off[v];
    f_row_off[v] = e < m ? kpos[e] : *m_kept;
}

// The source of every edge, from the tile schedule: one wave per tile, longer
// rows by workgroups.
__global__ void __launch_bounds__(kBlock) k_edge_sources(LongRows rows,
                                                         const uint4* __restrict__ tiles,
                                                         const uint32_t* __restrict__ act,
                                                         const uint32_t* __restrict__ act_off, uint32_t n_tiles,
                                                         uint32_t* __restrict__ src) {
    __shared__ struct {
        uint32_t v[kTileMaxVerts];
        alignas(8) uint8_t owner[kTileMaxEdges];
    } sh[kWaves];
    const uint32_t tid = threadIdx.x;
    if (blockIdx.x < rows.blocks()) {
        uint32_t e0, e1;
        const uint32_t v = rows.share(blockIdx.x, &e0, &e1);
        for (uint32_t e = e0 + tid; e < e1; e += kBlock) src[e] = v;
        return;
    }
    const uint32_t lane = lane_id(), tile = (blockIdx.x - rows.blocks()) * kWaves + (tid >> 6);
    if (tile >= n_tiles) return;
    auto& S = sh[tid >> 6];
    const uint4 td = tiles[tile];
    const uint32_t nv = td.y - td.x, ne = td.w - td.z;
    uint32_t off = 0;
    if (lane < nv) {
        S.v[lane] = act[td.x + lane];
        off = act_off[td.x + lane] - td.z;
    }
    tile_owners(S.owner, lane < nv, off);
    for (uint32_t j = lane; j < ne; j += 64) src[td.z + j] = S.v[S.owner[j]];
}

// The kept edges, in order.
template <typename LabT>
__global__ void __launch_bounds__(kBlock) k_kept_edges(const uint32_t* __restrict__ src,
                                                       const uint32_t* __restrict__ tgt,
                                                       const LabT* __restrict__ lab, uint32_t m,
                                                       const uint32_t* __restrict__ keep,
                                                       const uint32_t* __restrict__ kpos,
                                                       uint32_t* __restrict__ f_src, uint32_t* __restrict__ f_tgt,
                                                       LabT* __restrict__ f_lab) {
    const uint32_t e = blockIdx.x * kBlock + threadIdx.x;
    if (e >= m || !keep[e]) return;
    const uint32_t p = kpos[e];
    f_src[p] = src[e];
    f_tgt[p] = tgt[e];
    f_lab[p] = lab[e];
}

// Sort keys of the reversal: the target above the source and the label, or,
// where the three do not fit 64 bits, above the edge's number.
struct RevKey {
    int lab_bits, src_bits;  // both 0: the low 32 bits are the edge
    __host__ __device__ int low() const { return src_bits ? lab_bits + src_bits : 32; }
};

template <typename LabT>
__global__ void __launch_bounds__(kBlock) k_rev_keys(const uint32_t* __restrict__ src,
                                                     const uint32_t* __restrict__ tgt,
                                                     const LabT* __restrict__ lab, uint32_t m, RevKey rk,
                                                     uint64_t* __restrict__ keys) {
    const uint32_t e = blockIdx.x * kBlock + threadIdx.x;
    if (e >= m) return;
    const uint64_t rest = rk.src_bits ? (static_cast<uint64_t>(src[e]) << rk.lab_bits) | lab[e] : e;
    keys[e] = (static_cast<uint64_t>(tgt[e]) << rk.low()) | rest;
}

// first[w] = position of the first sorted key with target >= w, w = 0..n.
// An edge writes the entries of the targets between its predecessor's and its
// own, up to kRevGap of them; the rest of a longer gap (a graph whose edges
// end in few vertices) keeps kNoFirst and is searched entry by entry.
constexpr uint32_t kRevGap = 64, kNoFirst = 0xFFFFFFFFu;

__global__ void __launch_bounds__(kBlock) k_rev_first(const uint64_t* __restrict__ keys, uint32_t m, uint32_t n,
                                                      int low, uint32_t* __restrict__ first) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i > m) return;
    const uint32_t lo = i ? static_cast<uint32_t>(keys[i - 1] >> low) + 1 : 0u;
    const uint32_t hi = i < m ? static_cast<uint32_t>(keys[i] >> low) : n;
    for (uint32_t w = lo; w <= hi && w - lo < kRevGap; w++) first[w] = i;
}

__global__ void __launch_bounds__(kBlock) k_rev_gaps(const uint64_t* __restrict__ keys, uint32_t m, uint32_t n,
                                                     int low, uint32_t* __restrict__ first) {
    const uint32_t w = blockIdx.x * kBlock + threadIdx.x;
    if (w > n || first[w] != kNoFirst) return;
    uint32_t lo = 0, hi = m;
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (static_cast<uint32_t>(keys[mid] >> low) < w) lo = mid + 1; else hi = mid;
    }
    first[w] = lo;
}

// Row offsets of h: with both directions a row holds the vertex's kept
// out-edges, then its kept in-edges.
__global__ void __launch_bounds__(kBlock) k_both_rows(const uint32_t* __restrict__ f_row_off,
                                                      const uint32_t* __restrict__ first, uint32_t n,
                                                      uint32_t* __restrict__ h_row_off) {
    const uint32_t v = blockIdx.x * kBlock + threadIdx.x;
    if (v <= n) h_row_off[v] = f_row_off[v] + first[v];
}

// Each kept edge (v, l, w) as the edge (w, l + label_add, v) of row w: sorted
// key i goes to position i, past the out-edges of rows 0..w with both
// directions (f_row_off set).
template <typename LabT>
__global__ void __launch_bounds__(kBlock) k_rev_edges(const uint64_t* __restrict__ keys, uint32_t m, RevKey rk,
                                                      const uint32_t* __restrict__ f_src,
                                                      const LabT* __restrict__ f_lab,
                                                      const uint32_t* __restrict__ f_row_off, uint32_t label_add,
                                                      uint32_t* __restrict__ h_tgt, uint32_t* __restrict__ h_lab) {
    const uint32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= m) return;
    const uint64_t k = keys[i];
    const uint32_t w = static_cast<uint32_t>(k >> rk.low());
    uint32_t v, l;
    if (rk.src_bits) {
        v = static_cast<uint32_t>(k >> rk.lab_bits) & ((1u << rk.src_bits) - 1);
        l = static_cast<uint32_t>(k) & ((1u << rk.lab_bits) - 1);
    } else {
        v = f_src[static_cast<uint32_t>(k)];
        l = static_cast<uint32_t>(f_lab[static_cast<uint32_t>(k)]);
    }
    const uint32_t p = f_row_off ? f_row_off[w + 1] + i : i;
    h_tgt[p] = v;
    h_lab[p] = l + label_add;
}

// The kept out-edges in their rows of h: before edge e lie the in-edges of
// the rows before its own.
template <typename LabT>
__global__ void __launch_bounds__(kBlock) k_copy_out(const uint32_t* __restrict__ f_src,
                                                     const uint32_t* __restrict__ f_tgt,
                                                     const LabT* __restrict__ f_lab, uint32_t m,
                                                     const uint32_t* __restrict__ first,
                                                     uint32_t* __restrict__ h_tgt, uint32_t* __restrict__ h_lab) {
    const uint32_t e = blockIdx.x * kBlock + threadIdx.x;
    if (e >= m) return;
    const uint32_t p = first[f_src[e]] + e;
    h_tgt[p] = f_tgt[e];
    h_lab[p] = static_cast<uint32_t>(f_lab[e]);
}

template <typename LabT>
void build_view(const Staged& g, uint32_t flags, const std::vector<uint32_t>* labels, DirectedView& out,
                Arena& arena, hipStream_t s) {
    const uint32_t n = g.n, m = static_cast<uint32_t>(g.m);
    const LabT* lab = static_cast<const LabT*>(g.lab);
    const bool reversed = (flags & (BSIM_BACKWARD | BSIM_BOTH_DIRECTIONS)) != 0;
    Staged& f = out.f;
    f = g;
    out.f_staged = true;
    uint32_t* src = arena.alloc<uint32_t>(static_cast<size_t>(m) + 1);
    if (m)
        k_edge_sources<<<long_rows(g).blocks() + ceil_div(g.n_tiles, kWaves), kBlock, 0, s>>>(
            long_rows(g), g.tiles, g.act, g.act_off, g.n_tiles, src);
    uint32_t m_f = m;
    if (labels) {
        // the kept edges
        const uint32_t mask_size = g.max_label + 1;
        uint8_t* mask = arena.alloc<uint8_t>(mask_size);
        hip_check(hipMemsetAsync(mask, 0, mask_size, s), "label mask");
        if (!labels->empty()) {
            uint32_t* ids = arena.alloc<uint32_t>(labels->size());
            hip_check(hipMemcpyAsync(ids, labels->data(), labels->size() * 4, hipMemcpyHostToDevice, s),
                      "label set");
            const uint32_t ni = static_cast<uint32_t>(labels->size());
            k_label_mask<<<ceil_div(ni, kBlock), kBlock, 0, s>>>(ids, ni, mask, mask_size);
        }
        uint32_t* keep = arena.alloc<uint32_t>(static_cast<size_t>(m) + 1);
        uint32_t* kpos = arena.alloc<uint32_t>(static_cast<size_t>(m) + 1);
        uint32_t* total = arena.alloc<uint32_t>(1);
        uint32_t* f_row_off = arena.alloc<uint32_t>(static_cast<size_t>(n) + 1);
        if (m) k_keep_flags<LabT><<<ceil_div(m, kBlock), kBlock, 0, s>>>(lab, m, mask, keep);
        scan_exclusive(keep, kpos, m, total, arena, s);
        k_kept_rows<<<ceil_div(static_cast<uint64_t>(n) + 1, kBlock), kBlock, 0, s>>>(g.row_off, n, m, kpos, total,
                                                                                      f_row_off);
        hip_check(hipMemcpyAsync(&m_f, total, 4, hipMemcpyDeviceToHost, s), "kept edge count");
        hip_check(hipStreamSynchronize(s), "kept edge count");
        uint32_t* f_src = arena.alloc<uint32_t>(static_cast<size_t>(m_f) + 1);
        uint32_t* f_tgt = arena.alloc<uint32_t>(static_cast<size_t>(m_f) + 1);
        LabT* f_lab = arena.alloc<LabT>(static_cast<size_t>(m_f) + 1);
        if (m)
            k_kept_edges<LabT><<<ceil_div(m, kBlock), kBlock, 0, s>>>(src, g.tgt, lab, m, keep, kpos, f_src, f_tgt,
                                                                      f_lab);
        f = Staged{};
        f.n = n;
        f.m = m_f;
        f.label_bytes = g.label_bytes;
        f.row_off = f_row_off;
        f.tgt = f_tgt;
        f.lab = f_lab;
        f.type_off = g.type_off;
        f.type_ids = g.type_ids;
        f.alive = g.alive;
        f.max_label = g.max_label;
        f.hub_table_slots = g.hub_table_slots;
        f.trusted = true;
        out.f_staged = false;
        src = f_src;
    }
    hip_check(hipGetLastError(), "kept edges");
    Staged& h = out.h;
    if (!reversed) {
        h = f;
        return;
    }
    const bool both = (flags & BSIM_BOTH_DIRECTIONS) != 0;
    const uint64_t m_h = both ? 2ull * m_f : m_f;
    if (m_h >= (1ull << 32))
        throw DeviceError{BSIM_E_UNSUPPORTED, "both edge directions together reach 2^32 edges"};
    const uint32_t L = g.max_label + 1;
    if (both && L > (1u << 24)) throw DeviceError{BSIM_E_UNSUPPORTED, "edge labels must be < 2^24"};
    const LabT* f_lab = static_cast<const LabT*>(f.lab);
    const int vbits = std::max(1, bit_width(n ? n - 1 : 0)), lbits = std::max(1, bit_width(g.max_label));
    const RevKey rk = 2 * vbits + lbits <= 64 && vbits < 32 ? RevKey{lbits, vbits} : RevKey{0, 0};
    uint64_t* keys = arena.alloc<uint64_t>(static_cast<size_t>(m_f) + 1);
    uint64_t* keys2 = arena.alloc<uint64_t>(static_cast<size_t>(m_f) + 1);
    uint32_t* first = arena.alloc<uint32_t>(static_cast<size_t>(n) + 1);
    uint32_t* h_row_off = both ? arena.alloc<uint32_t>(static_cast<size_t>(n) + 1) : first;
    uint32_t* h_tgt = arena.alloc<uint32_t>(m_h + 1);
    uint32_t* h_lab = arena.alloc<uint32_t>(m_h + 1);
    const uint32_t gm = std::max<uint32_t>(ceil_div(m_f, kBlock), 1);
    if (m_f) {
        k_rev_keys<LabT><<<gm, kBlock, 0, s>>>(src, f.tgt, f_lab, m_f, rk, keys);
        keys = radix_sort(keys, keys2, m_f, rk.low() + vbits, arena, s, rk.low());
    }
    const uint32_t gn = ceil_div(static_cast<uint64_t>(n) + 1, kBlock);
    hip_check(hipMemsetAsync(first, 0xFF, (static_cast<size_t>(n) + 1) * 4, s), "reversed rows");
    k_rev_first<<<ceil_div(static_cast<uint64_t>(m_f) + 1, kBlock), kBlock, 0, s>>>(keys, m_f, n, rk.low(), first);
    k_rev_gaps<<<gn, kBlock, 0, s>>>(keys, m_f, n, rk.low(), first);
    if (both) k_both_rows<<<gn, kBlock, 0, s>>>(f.row_off, first, n, h_row_off);
    if (m_f) {
        k_rev_edges<LabT><<<gm, kBlock, 0, s>>>(keys, m_f, rk, src, f_lab, both ? f.row_off : nullptr, both ? L : 0u,
                                                h_tgt, h_lab);
        if (both) k_copy_out<LabT><<<gm, kBlock, 0, s>>>(src, f.tgt, f_lab, m_f, first, h_tgt, h_lab);
    }
    hip_check(hipGetLastError(), "direction view");
    h = Staged{};
    h.n = n;
    h.m = m_h;
    h.label_bytes = 4;
    h.row_off = h_row_off;
    h.tgt = h_tgt;
    h.lab = h_lab;
    h.type_off = g.type_off;
    h.type_ids = g.type_ids;
    h.alive = g.alive;
    h.hub_table_slots = g.hub_table_slots;
    h.max_label = both ? 2 * L - 1 : g.max_label;
    h.in_label_base = both ? L : 0;
    h.trusted = true;
}

}  // namespace

void direction_view(const Staged& g, uint32_t flags, const std::vector<uint32_t>* labels, bool want_edges,
                    DirectedView& out, StageHost* host, Arena& arena, hipStream_t s) {
    if (g.label_bytes == 2)
        build_view<uint16_t>(g, flags, labels, out, arena, s);
    else
        build_view<uint32_t>(g, flags, labels, out, arena, s);
    stage_graph(out.h, host, arena, s);
    if (out.f_staged) return;
    // the kept edges need a schedule of their own only for the summary edges
    if (!(flags & (BSIM_BACKWARD | BSIM_BOTH_DIRECTIONS)))
        out.f = out.h;
    else if (want_edges)
        stage_graph(out.f, host, arena, s);
}

}  // namespace bsim

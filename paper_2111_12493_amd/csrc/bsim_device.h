// bsim_device.h -- device helpers shared by the refinement and finalize
// kernels: wave64 reductions, the open-addressing count table, and the tile
// layout (which vertex of a tile owns each edge).
#pragma once

#include "bsim_internal.h"

namespace bsim {

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63; }

// salt(l) = M(C_L + l); at and past in_base (when nonzero) the salts of
// incoming edges: label in_base + l is salted as label l + 2^31.
__device__ __forceinline__ uint64_t label_salt(uint32_t l, uint32_t in_base) {
    return mix64(kCL + ((in_base && l >= in_base) ? 0x80000000ull + (l - in_base) : static_cast<uint64_t>(l)));
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t x, int d) {
    uint32_t lo = static_cast<uint32_t>(__shfl_xor(static_cast<int>(static_cast<uint32_t>(x)), d, 64));
    uint32_t hi = static_cast<uint32_t>(__shfl_xor(static_cast<int>(static_cast<uint32_t>(x >> 32)), d, 64));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += static_cast<uint32_t>(__shfl_xor(static_cast<int>(x), d, 64));
    return x;
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t x) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += shfl_xor_u64(x, d);
    return x;
}

// Sum over the block; valid in thread 0.  `red` needs kBlock/64 entries.
__device__ __forceinline__ uint32_t block_sum_u32(uint32_t x, uint32_t* red) {
    x = wave_sum_u32(x);
    if (lane_id() == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    uint32_t t = 0;
    if (threadIdx.x == 0)
        for (int i = 0; i < kBlock / 64; i++) t += red[i];
    __syncthreads();
    return t;
}

__device__ __forceinline__ uint64_t block_sum_u64(uint64_t x, uint64_t* red) {
    x = wave_sum_u64(x);
    if (lane_id() == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    uint64_t t = 0;
    if (threadIdx.x == 0)
        for (int i = 0; i < kBlock / 64; i++) t += red[i];
    __syncthreads();
    return t;
}

// Current value of an LDS table slot other lanes may be writing.  A relaxed
// atomic load (a volatile one would keep the generic address space and
// compile to a flat load, which also waits on every global load in flight).
__device__ __forceinline__ uint64_t lds_peek(uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Insert a nonzero key into an LDS open-addressing region; returns 1 if it
// was not present.  A slot only changes from 0 to a key while it is in use, so
// it is read before it is CASed: the read sees the key (no atomic needed), or a
// 0 that the CAS then resolves.
__device__ __forceinline__ uint32_t lds_insert(uint64_t* tab, uint32_t slot, uint32_t base,
                                               uint32_t end, uint64_t f) {
    for (;;) {
        uint64_t cur = lds_peek(&tab[slot]);
        if (cur == f) return 0u;
        if (cur == 0) {
            unsigned long long old = atomicCAS(reinterpret_cast<unsigned long long*>(&tab[slot]), 0ull,
                                               static_cast<unsigned long long>(f));
            if (old == 0ull) return 1u;
            if (old == f) return 0u;
        }
        if (++slot == end) slot = base;
    }
}

// Insert a nonzero key into an LDS table of `slots` slots, probing at most
// `slots` positions: 1 = inserted, 0 = already present, 2 = table full.
__device__ __forceinline__ uint32_t lds_insert_bounded(uint64_t* tab, uint32_t slot, uint32_t slots,
                                                       uint64_t f) {
    for (uint32_t step = 0; step < slots; step++) {
        uint64_t cur = lds_peek(&tab[slot]);
        if (cur == f) return 0u;
        if (cur == 0) {
            unsigned long long old = atomicCAS(reinterpret_cast<unsigned long long*>(&tab[slot]), 0ull,
                                               static_cast<unsigned long long>(f));
            if (old == 0ull) return 1u;
            if (old == f) return 0u;
        }
        if (++slot == slots) slot = 0;
    }
    return 2u;
}

// Order the LDS accesses of one wave: its LDS operations execute in program
// order, so only the compiler has to be held.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// x of the lane that the DPP control names, 0 where there is none or the
// lane's row is not in kRows.
template <int kCtrl, int kRows>
__device__ __forceinline__ uint32_t dpp_or_0(uint32_t x) {
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), kCtrl, kRows, 0xf, false));
}
template <int kCtrl, int kRows>
__device__ __forceinline__ uint64_t dpp_or_0(uint64_t x) {
    return (static_cast<uint64_t>(dpp_or_0<kCtrl, kRows>(static_cast<uint32_t>(x >> 32))) << 32) |
           dpp_or_0<kCtrl, kRows>(static_cast<uint32_t>(x));
}

// Inclusive sum over the 64 lanes in registers: four shifts within the rows
// of 16 lanes, then the totals of row 0 and 2 to the next row, then that of
// the lower half to the upper.
template <typename T>
__device__ __forceinline__ T wave_incl_sum(T x) {
    x += dpp_or_0<0x111, 0xf>(x);
    x += dpp_or_0<0x112, 0xf>(x);
    x += dpp_or_0<0x114, 0xf>(x);
    x += dpp_or_0<0x118, 0xf>(x);
    x += dpp_or_0<0x142, 0xa>(x);
    x += dpp_or_0<0x143, 0xc>(x);
    return x;
}

// Which vertex of a tile owns each of a lane's kLaneEdges consecutive edges
// (lane l holds local edges [l kLaneEdges, (l + 1) kLaneEdges)).  Lane i < nv
// passes the first local edge of vertex i; every vertex of a tile has edges.
// `marks` is kTileMaxEdges bytes of the wave's LDS, 8-byte aligned, free
// again on return.
struct LaneOwners {
    uint64_t starts;   // byte q: 1 if edge q of this lane begins a vertex
    uint32_t before;   // vertices that begin in earlier lanes
    // local vertex of edge q (q known at compile time)
    __device__ __forceinline__ uint32_t of(int q) const {
        const uint64_t upto = q == 7 ? starts : starts & ((1ull << (8 * (q + 1))) - 1);
        return before + static_cast<uint32_t>(__popcll(upto)) - 1;
    }
    __device__ __forceinline__ bool begins(int q) const { return (starts >> (8 * q)) & 1; }
};
__device__ __forceinline__ LaneOwners lane_owners(uint8_t* marks, bool mine, uint32_t off) {
    static_assert(kLaneEdges == 8, "one 8-byte word of marks per lane");
    uint64_t* word = reinterpret_cast<uint64_t*>(marks) + lane_id();
    *word = 0;
    wave_sync();
    if (mine) marks[off] = 1;
    wave_sync();
    LaneOwners o;
    o.starts = *word;
    wave_sync();
    const uint32_t c = static_cast<uint32_t>(__popcll(o.starts));
    o.before = wave_incl_sum(c) - c;
    return o;
}

// The same as a byte per local edge in LDS (owner[j], kTileMaxEdges bytes),
// for kernels that walk a tile's edges lane by lane.
__device__ __forceinline__ void tile_owners(uint8_t* owner, bool mine, uint32_t off) {
    const LaneOwners o = lane_owners(owner, mine, off);
    uint64_t word = 0;
#pragma unroll
    for (int q = 0; q < kLaneEdges; q++) word |= static_cast<uint64_t>(o.of(q) & 0xFF) << (8 * q);
    reinterpret_cast<uint64_t*>(owner)[lane_id()] = word;
    wave_sync();
}

}  // namespace bsim

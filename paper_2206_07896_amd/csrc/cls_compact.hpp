// cls_compact.hpp -- tile body of the COMPACT_I32 class: stream compaction
// (a database selection), y = the elements of x greater than t, in order,
// count = how many.
//
// A tile is B threads x I items, B*I consecutive elements; 32-lane warp w
// owns the consecutive segment [w*32*I, (w+1)*32*I) of it.
//   1. local offsets, by warp vote.  With I >= 4 a tile is read in rows of 32
//      lanes x 4 elements (16 bytes per lane, at any alignment) and held in
//      registers.  A lane keeps c = 0..4 of its four; the three bit planes
//      of c are balloted over the warp, and popc of each plane below the lane,
//      scaled by 2^plane, is the number kept by the lanes before it.  Rows are
//      chained by their totals.  Smaller I take one element per lane per step
//      (one ballot, popc below the lane), in two passes over the tile (count,
//      then place).
//   2. warp totals through LDS; barrier; each warp's offset in the tile and
//      the tile's count;
//   3. the tile's offset in y by decoupled look-back over the tiles' counts
//      (the scan class's protocol: tiles start in ticket order);
//   4. before the look-back, every kept element is written to an LDS stage
//      at warp offset + its own (the tile's output, contiguous); after it,
//      the block copies the stage to y at the tile's offset with coalesced
//      stores.
// The tile in which x ends is another matter (compact_end): guards on the rows
// of every tile cost the kernel 23 registers and its full tiles 3%, one element
// per lane and step through a last tile of 1024 x 32 10 us.
// The last tile writes count.  The pieces below are sequenced by the
// kernel (k_compact.hip), which overlaps one tile's look-back and copy-out
// with the next tile's loads and count.
#pragma once
#include "cls_scan.hpp"

namespace spmd {

template <int B, int I>
struct CompactLds {
    uint32_t warp[B / 32];
    uint32_t excl;
    uint32_t stage[B * I];  // the tile's kept elements, in order
};

// number of lanes below this one in the half-wave whose bit is set in m
__device__ __forceinline__ uint32_t below(uint32_t m) {
    return (uint32_t)__builtin_popcount(m & ((1u << lane32()) - 1u));
}

// A tile between its loads and its stage: the rows it holds in registers
// (rows form only) and each lane's kept-before count per row.
template <int B, int I>
struct CompactFront {
    static constexpr int S = I >= 4 ? I / 4 : 1;
    u32x4 rv[S];
    uint32_t rpos[S];  // kept elements of this warp's segment before this lane's four
};

// Issue a full tile's loads (rows form, 16 bytes per lane at any alignment;
// smaller items load in the two passes).
template <int B, int I>
__device__ __forceinline__ void compact_issue(const int32_t* __restrict__ x, uint32_t tile, CompactFront<B, I>& F) {
    if constexpr (I >= 4) {
        const u32x4_a4* xv = reinterpret_cast<const u32x4_a4*>(x + (uint64_t)tile * B * I +
                                                               (uint64_t)(threadIdx.x >> 5) * 32u * I);
#pragma unroll
        for (int q = 0; q < F.S; ++q) F.rv[q] = __builtin_nontemporal_load(xv + q * 32 + lane32());
    }
}

// The lane's kept count before each of its four elements of a row, and the
// row's total.
__device__ __forceinline__ uint32_t compact_row(const u32x4& v, int32_t t, uint32_t& total) {
    const uint32_t c = ((int32_t)v.x > t) + ((int32_t)v.y > t) + ((int32_t)v.z > t) + ((int32_t)v.w > t);
    const uint32_t m0 = w32_ballot(c & 1u), m1 = w32_ballot(c & 2u), m2 = w32_ballot(c & 4u);
    total = (uint32_t)__builtin_popcount(m0) + 2u * (uint32_t)__builtin_popcount(m1) +
            4u * (uint32_t)__builtin_popcount(m2);
    return below(m0) + 2u * below(m1) + 4u * below(m2);
}

// Step 1: local offsets by warp vote; lane 0 of each warp writes the
// warp's count to LDS (the caller then places a barrier).
template <int B, int I>
__device__ __forceinline__ void compact_count(const int32_t* __restrict__ x, uint32_t n, int32_t t, uint32_t tile,
                                              CompactFront<B, I>& F, CompactLds<B, I>& L) {
    uint32_t run = 0;  // warp-uniform
    if constexpr (I >= 4) {
#pragma unroll
        for (int q = 0; q < F.S; ++q) {
            uint32_t total;
            F.rpos[q] = run + compact_row(F.rv[q], t, total);
            run += total;
        }
    } else {
        const uint64_t seg = (uint64_t)tile * B * I + (uint64_t)(threadIdx.x >> 5) * 32u * I;
        for (int k = 0; k < I; ++k) {
            const uint64_t e = seg + (uint64_t)k * 32u + lane32();
            const bool keep = e < (uint64_t)n && x[e] > t;
            run += (uint32_t)__builtin_popcount(w32_ballot(keep));
        }
    }
    if (lane32() == 0) L.warp[threadIdx.x >> 5] = run;
}

// Step 2 (after the barrier): the tile's count and this warp's offset in it.
template <int B, int I>
__device__ __forceinline__ void compact_sums(const CompactLds<B, I>& L, uint32_t& agg, uint32_t& wpre) {
    constexpr int NW = B / 32;
    const uint32_t w = threadIdx.x >> 5;
    agg = 0;
    wpre = 0;
#pragma unroll 8  // all 32 at once took the registers to 126, with spills, and 3% of the time
    for (int k = 0; k < NW; ++k) {
        const uint32_t s = L.warp[k];
        agg += s;
        wpre += ((uint32_t)k < w) ? s : 0u;
    }
}

// Step 4, first half: every kept element to the LDS stage at its offset in
// the tile's output.
template <int B, int I>
__device__ __forceinline__ void compact_stage(const int32_t* __restrict__ x, uint32_t n, int32_t t, uint32_t tile,
                                              uint32_t wpre, const CompactFront<B, I>& F, CompactLds<B, I>& L) {
    if constexpr (I >= 4) {
#pragma unroll
        for (int q = 0; q < F.S; ++q) {
            uint32_t p = wpre + F.rpos[q];
            const uint32_t v[4] = {F.rv[q].x, F.rv[q].y, F.rv[q].z, F.rv[q].w};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((int32_t)v[j] > t) L.stage[p++] = v[j];
        }
        return;
    }
    const uint64_t seg = (uint64_t)tile * B * I + (uint64_t)(threadIdx.x >> 5) * 32u * I;
    uint32_t p = wpre;  // warp-uniform
    for (int k = 0; k < I; ++k) {
        const uint64_t e = seg + (uint64_t)k * 32u + lane32();
        const int32_t v = e < (uint64_t)n ? x[e] : 0;
        const bool keep = e < (uint64_t)n && v > t;
        const uint32_t m = w32_ballot(keep);
        if (keep) L.stage[p + below(m)] = (uint32_t)v;
        p += (uint32_t)__builtin_popcount(m);
    }
}

// The tile in which x ends: no other tile waits for it, so it looks back first
// and then takes pieces of 8 (or 4) elements per thread one after another, rows
// of 32 lanes x 4 straight from registers to y.  Past n a row holds the least
// value, which no t lets through.
template <int B, int I>
__device__ __forceinline__ void compact_end(const int32_t* __restrict__ x, int32_t* __restrict__ y, uint32_t* count,
                                            uint32_t n, int32_t t, uint32_t tile, uint64_t* status, uint32_t tag,
                                            uint32_t* err, CompactLds<B, I>& L) {
    constexpr int S = I >= 8 ? 2 : 1;
    const uint32_t tid = threadIdx.x;
    if (tid < 64) {
        const uint32_t excl = scan_lookback(status, tile, 0u, tag, err, true);
        if (tid == 0) L.excl = excl;
    }
    __syncthreads();
    uint32_t run = L.excl;
#pragma unroll 1
    for (uint64_t base = (uint64_t)tile * B * I; base < (uint64_t)n; base += 4ull * S * B) {
        const uint64_t e0 = base + (uint64_t)(tid >> 5) * 128u * S + 4u * lane32();
        u32x4 v[S];
        uint32_t pos[S], mine = 0;
#pragma unroll
        for (int q = 0; q < S; ++q) {
            const uint64_t e = e0 + 128u * q;
            v[q] = u32x4{0x80000000u, 0x80000000u, 0x80000000u, 0x80000000u};
            if (e + 4 <= (uint64_t)n) {
                v[q] = *reinterpret_cast<const u32x4_a4*>(x + e);
            } else {
                if (e < (uint64_t)n) v[q].x = (uint32_t)x[e];
                if (e + 1 < (uint64_t)n) v[q].y = (uint32_t)x[e + 1];
                if (e + 2 < (uint64_t)n) v[q].z = (uint32_t)x[e + 2];
            }
        }
#pragma unroll
        for (int q = 0; q < S; ++q) {
            uint32_t total;
            pos[q] = mine + compact_row(v[q], t, total);
            mine += total;
        }
        if (lane32() == 0) L.warp[tid >> 5] = mine;
        __syncthreads();
        uint32_t agg, wpre;
        compact_sums<B, I>(L, agg, wpre);
        __syncthreads();  // the next piece writes L.warp
#pragma unroll
        for (int q = 0; q < S; ++q) {
            int32_t* yo = y + run + wpre + pos[q];
            const uint32_t w[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((int32_t)w[j] > t) *yo++ = (int32_t)w[j];
        }
        run += agg;
    }
    if (tid == 0) *count = run;
}

}  // namespace spmd

// cls_jacobi.hpp -- body of the JACOBI5_F32 class: one sweep of the 5-point
// Laplace-Jacobi stencil.
//
// A wave owns a strip of up to 256 columns (64 lanes x 4) and R rows, in
// registers: it loads the R rows and the one above and below, 16 bytes per
// lane at any alignment, and one element beside each row's ends; north and
// south neighbours are the lane's own registers, west and east the adjacent
// lanes' (DPP wave shifts).  Every cell is 0.25f * ((N + S) + (W + E)) with each
// operation rounded to fp32 in that order (no contraction); border cells are
// copied.  Cells outside the grid are neither read nor stored.
//
// All loads of a strip are in flight at once and nothing is shared between
// waves, so there is no LDS tile, no barrier, and one body for every block
// shape, width and alignment.  Bound by memory.  A sweep on buffers that no cache
// holds: 2001 x 1999 6.1 us, 8.2 with an LDS tile that four 4-byte loads per thread
// and row filled; 4099 x 4001 27.7 us against 30.2; 8190 x 8191 89.5 against 101;
// 8192^2 84.4 us (6.4 TB/s) against 86.5 with a tile that 16-byte loads filled.
#pragma once
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "warp32.hpp"

namespace spmd {

// Workgroups are dealt to the 8 XCDs round-robin by linear id, and each XCD
// has its own L2.  Tile t of XCD x = id mod 8 is the (id / 8)-th of a
// contiguous range of tiles, so neighbouring tiles -- which read each
// other's edge lines as halo -- run on the same XCD and share its L2.
constexpr uint32_t NUM_XCD = 8;

__device__ __forceinline__ uint32_t xcd_tile(uint32_t id, uint32_t nt) {
    const uint32_t q = nt / NUM_XCD, r = nt % NUM_XCD;
    const uint32_t x = id % NUM_XCD, local = id / NUM_XCD;
    return x < r ? x * (q + 1) + local : r * (q + 1) + (x - r) * q + local;
}

// Launch grid of gx x gy tiles, which blocks find by their linear id (t % gx,
// t / gx).  A grid's y ends at 65536, so taller ones are folded into x; the last
// tiles may then lie below the grid.
inline dim3 tile_grid(uint64_t gx, uint64_t gy) {
    const uint64_t fold = (gy + 65535) / 65536;
    return dim3((uint32_t)(gx * fold), (uint32_t)((gy + fold - 1) / fold));
}

constexpr int JS_W = 256;  // columns of a strip

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes at any float's address

// f(0), ..., f(N - 1) with the index a constant.  A loop over rows held in
// registers is unrolled late, after an array of up to 32 of them has been taken
// for one vector and copied whole on every write (short bands spilled).
template <typename F, int... I>
__device__ __forceinline__ void each_row(F f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void each_row(F f) {
    each_row(f, std::make_integer_sequence<int, N>{});
}

// The value of the lane to the left (right); lane 0 (63) gets `end`.
__device__ __forceinline__ float lane_left(float v, float end) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(end), __float_as_int(v), 0x138, 0xf, 0xf, false));  // wave_shr:1
}
__device__ __forceinline__ float lane_right(float v, float end) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(end), __float_as_int(v), 0x130, 0xf, 0xf, false));  // wave_shl:1
}

// Four columns from 16 bytes that end at the row's last element, where the row
// ends `over` (1..3) elements into them: the elements move down, what is past
// the end is never used.
__device__ __forceinline__ f32x4 row_end(f32x4 t, int64_t over) {
    f32x4 c = t;
    c.x = over == 1 ? t.y : over == 2 ? t.z : t.w;
    c.y = over == 1 ? t.z : t.w;
    c.z = t.w;
    return c;
}

// As jacobi_strip, for grids of one to three columns: a lane per cell.
template <int R>
__device__ __forceinline__ void jacobi_thin(const float* __restrict__ u, float* __restrict__ v, int64_t NX, int64_t NY,
                                            int64_t y0) {
#pragma clang fp contract(off)
    const int64_t gx = lane64() % NX, gy = y0 + lane64() / NX;
    if (gy >= NY || gy >= y0 + R) return;
    const float* p = u + gy * NX + gx;
    float o = p[0];
    if (gx > 0 && gx < NX - 1 && gy > 0 && gy < NY - 1) o = 0.25f * ((p[-NX] + p[NX]) + (p[-1] + p[1]));
    v[gy * NX + gx] = o;
}

// One wave: columns [x0, xe), xe <= x0 + 256, of rows [y0, min(y0 + R, NY)),
// y0 < NY.  xe is NX or x0 plus a multiple of 4.  KEEP: v is read again soon.
template <int R, bool KEEP = false>
__device__ __forceinline__ void jacobi_strip(const float* __restrict__ u, float* __restrict__ v, int64_t NX, int64_t NY,
                                             int64_t x0, int64_t xe, int64_t y0) {
#pragma clang fp contract(off)
    static_assert(3 * R <= 64, "a lane per cell of a thin grid");
    if (NX < 4) return jacobi_thin<R>(u, v, NX, NY, y0);
    const int lane = (int)lane64();
    const int64_t gx = x0 + 4 * lane;
    // Lanes that own cells, and the one after them for its first cell.
    const bool in = gx < NX && gx <= xe;
    const bool full = gx + 4 <= NX;
    const int64_t origin = (y0 - 1) * NX + x0;
    const int above = y0 > 0 ? 0 : 1;                         // first row of 0 .. R + 1 that exists
    const int rows = NY - y0 < R ? (int)(NY - y0) : R;        // rows owned
    const int below = NY - y0 <= R ? (int)(NY - y0) : R + 1;  // last row that exists
    const int side = lane == 0 ? -1 : JS_W;                   // the element beside the strip
    const bool beside = (lane == 0 && x0 > 0) || (lane == 63 && x0 + JS_W < NX);
    const f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
    const int at = (int)(full ? 4 * lane : NX - 4 - x0);      // a lane that the row's end cuts: the row's last 16 bytes
    f32x4 c[R + 2];
    float end[R];
    each_row<R + 2>([&](auto row) __attribute__((always_inline)) {
        constexpr int i = row;
        c[i] = z;
        if constexpr (i >= 1 && i <= R) end[i - 1] = 0.0f;
        if (i >= above && i <= below) {  // wave-uniform
            const float* p = u + (origin + i * NX);
            if (in) c[i] = *reinterpret_cast<const f32x4_a4*>(p + at);
            if constexpr (i >= 1 && i <= R)
                if (beside) end[i - 1] = p[side];
        }
    });
    if ((NX & 3) && x0 + JS_W > NX)  // wave-uniform: the row ends inside a lane's four columns
        each_row<R + 2>([&](auto row) __attribute__((always_inline)) {
            constexpr int i = row;
            const f32x4 e = row_end(c[i], gx + 4 - NX);
            c[i] = full ? c[i] : e;
            __builtin_amdgcn_sched_barrier(0);
        });
    const bool own = gx < xe;
    const bool keep0 = gx <= 0 || gx >= NX - 1, keep1 = gx + 1 >= NX - 1, keep2 = gx + 2 >= NX - 1, keep3 = gx + 3 >= NX - 1;
    each_row<R>([&](auto row) __attribute__((always_inline)) {
        constexpr int i = row;
        if (i < rows) {
            const f32x4 cur = c[i + 1];
            const f32x4 ns = c[i] + c[i + 2];
            f32x4 we;
            we.x = lane_left(cur.w, end[i]) + cur.y;
            we.y = cur.x + cur.z;
            we.z = cur.y + cur.w;
            we.w = cur.z + lane_right(cur.x, end[i]);
            f32x4_a4 o = 0.25f * (ns + we);
            const bool same = y0 + i == 0 || y0 + i == NY - 1;
            o.x = keep0 || same ? cur.x : o.x;
            o.y = keep1 || same ? cur.y : o.y;
            o.z = keep2 || same ? cur.z : o.z;
            o.w = keep3 || same ? cur.w : o.w;
            float* p = v + (origin + (i + 1) * NX) + 4 * lane;
            // nontemporal: no part of this sweep reads v again (2001 x 1999
            // 6.6 us against 8.2, 8192^2 88 against 90)
            if (own && full) {
                if constexpr (KEEP) *reinterpret_cast<f32x4_a4*>(p) = o;
                else __builtin_nontemporal_store(o, reinterpret_cast<f32x4_a4*>(p));
            } else if (own) {
                p[0] = o.x;
                if (gx + 1 < NX) p[1] = o.y;
                if (gx + 2 < NX) p[2] = o.z;
            }
        }
    });
}

// As jacobi_strip for up to 64 columns, xe <= x0 + 64: a lane per column, since
// 64 columns would leave 47 of a strip's lanes idle, and lane 2i (2i + 1) reads
// the element before (after) row i for all.  Stores are plain: other waves
// write the rest of a line.
template <int R>
__device__ __forceinline__ void jacobi_narrow(const float* __restrict__ u, float* __restrict__ v, int64_t NX, int64_t NY,
                                              int64_t x0, int64_t xe, int64_t y0) {
#pragma clang fp contract(off)
    static_assert(2 * R <= 64, "a lane per element beside the strip");
    const int lane = (int)lane64();
    const int64_t gx = x0 + lane;
    const bool in = gx < NX;
    const int64_t origin = (y0 - 1) * NX + x0;
    const int above = y0 > 0 ? 0 : 1;
    const int rows = NY - y0 < R ? (int)(NY - y0) : R;
    const int below = NY - y0 <= R ? (int)(NY - y0) : R + 1;
    float c[R + 2], beside = 0.0f;
    each_row<R + 2>([&](auto row) __attribute__((always_inline)) {
        constexpr int i = row;
        c[i] = 0.0f;
        if (i >= above && i <= below && in) c[i] = u[origin + i * NX + lane];
    });
    if (lane < 2 * rows && ((lane & 1) ? x0 + 64 < NX : x0 > 0))
        beside = u[origin + (1 + (lane >> 1)) * NX + ((lane & 1) ? 64 : -1)];
    const bool own = gx < xe;
    const bool keep = gx == 0 || gx >= NX - 1;
    each_row<R>([&](auto row) __attribute__((always_inline)) {
        constexpr int i = row;
        if (i < rows) {
            const float cur = c[i + 1];
            const float west = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(beside), 2 * i));
            const float east = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(beside), 2 * i + 1));
            const float ns = c[i] + c[i + 2];
            const float we = lane_left(cur, west) + lane_right(cur, east);
            const float o = 0.25f * (ns + we);
            if (own) v[origin + (i + 1) * NX + lane] = keep || y0 + i == 0 || y0 + i == NY - 1 ? cur : o;
        }
    });
}

}  // namespace spmd

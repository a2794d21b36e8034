// cls_jacobi_tb.hpp -- block body of the JACOBI5T_F32 class: S sweeps of the
// 5-point Laplace-Jacobi stencil in one pass over HBM (temporal blocking).
//
// One sweep reads and writes every cell once, so a sweep-per-launch stencil
// is bound at 8 bytes per cell by HBM.  Here a workgroup loads a region of
// 256 columns x RS * WV rows -- its interior tile and a halo of S rows and
// HC >= S columns on each side -- runs S sweeps on it, and writes back only
// the interior: HBM moves about 8 bytes per cell per S sweeps, plus the halo.
//
// The region lives in registers.  A wave spans a whole region row (64
// lanes x 4 columns); the WV waves own bands of RS consecutive rows, each
// lane its 4 columns of every row of its band.  In a sweep, north and south
// neighbours come from the lane's own registers, west and east from the
// adjacent lanes (DPP wave shifts, folded into the additions), and only the
// first and last row of each band go through LDS to the neighbouring waves
// (two slots per sweep parity, one barrier per sweep).
//
// Phases:
//   load   the region row by row, 16 bytes per lane; cells outside the grid
//          are zero (a cell that is updated never reads them);
//   sweep  S times: publish the band's edge rows; barrier; read the
//          neighbours' edge rows; update the band top-down.  A cell is
//          updated as 0.25f * ((N + S) + (W + E)), each operation rounded
//          to fp32 in that order (no contraction), exactly as the one-sweep
//          class; border cells of the grid keep their value.  Every row of
//          the region is updated in every sweep: the outer ring, whose outer
//          neighbours do not exist, goes stale by one cell per sweep and
//          after S sweeps is still outside the interior;
//   store  the interior, cells inside the grid.
// Results are bit-identical to S sweeps of the one-sweep class.
//
// Four vector operations per cell and sweep and nothing else in the loop: the
// region inside the grid has a body of its own without border tests, and rows
// are kept apart (sched_barrier), which holds a 12-row band at 71 registers
// and three blocks of eight waves on a CU.  8 sweeps of 8192^2: 106 us, 5.0
// TB/s of the bytes that one pass needs (the bound is HBM, 87 us, behind it
// the vector unit, 70 us); 169 us with neighbours exchanged through the LDS
// pipe, a border test per cell, and 64-row tiles of 152 registers.  8 sweeps
// of a small grid (192 x 74): 5.2 us, 18.8 before.
#pragma once
#include "cls_jacobi.hpp"

namespace spmd {

constexpr int JT_W = 256;         // columns of a region
constexpr int JT_MAX_SWEEPS = 11;  // fused at most (the smallest region is 24 rows)

template <int WV>
struct JacobiTbLds {
    f32x4 edge[2][2][WV][64];  // [sweep parity][first row, last row][wave][lane]
};

// S sweeps of the band in `c`.  EDGE: the region holds border cells of the
// grid: `keep` marks this lane's border columns, and rows `top` and `bottom`
// of the band (outside 0..RS-1 if not in it) are border rows.
template <int RS, int WV, bool EDGE>
__device__ __forceinline__ void jacobi_tb_sweeps(f32x4 (&c)[RS], uint32_t sweeps, int w, int lane,
                                                 const bool (&keep)[4], int top, int bottom, JacobiTbLds<WV>& L) {
#pragma clang fp contract(off)
    const int wu = w > 0 ? w - 1 : 0, wd = w < WV - 1 ? w + 1 : w;  // the outer bands read a row that nothing needs
#pragma unroll 1
    for (uint32_t s = 0; s < sweeps; ++s) {
        const int par = (int)(s & 1u);
        L.edge[par][0][w][lane] = c[0];
        L.edge[par][1][w][lane] = c[RS - 1];
        __syncthreads();
        const f32x4 up = L.edge[par][1][wu][lane], dn = L.edge[par][0][wd][lane];
        f32x4 ns = up + c[1];
        each_row<RS>([&](auto row) __attribute__((always_inline)) {
            constexpr int i = row;
            const f32x4 cur = c[i];
            f32x4 ns_next = cur;
            if constexpr (i + 2 < RS) ns_next += c[i + 2];
            else ns_next += dn;
            f32x4 we;
            we.x = lane_left(cur.w, 0.0f) + cur.y;
            we.y = cur.x + cur.z;
            we.z = cur.y + cur.w;
            we.w = cur.z + lane_right(cur.x, 0.0f);
            f32x4 o = 0.25f * (ns + we);
            if constexpr (EDGE) {
                const bool same = i == top || i == bottom;  // wave-uniform
                o.x = keep[0] || same ? cur.x : o.x;
                o.y = keep[1] || same ? cur.y : o.y;
                o.z = keep[2] || same ? cur.z : o.z;
                o.w = keep[3] || same ? cur.w : o.w;
            }
            c[i] = o;
            ns = ns_next;
            __builtin_amdgcn_sched_barrier(0);
        });
    }
}

// One region whose first row and column are y0 and x0.  EDGE: part of it may
// lie outside the grid or on its border.
template <int RS, int WV, bool VEC, bool NT, bool EDGE>
__device__ __forceinline__ void jacobi_tb_region(const float* __restrict__ u, float* __restrict__ v, int64_t NX,
                                                 int64_t NY, uint32_t sweeps, uint32_t hc, int64_t x0, int64_t y0,
                                                 JacobiTbLds<WV>& L) {
    const int lane = (int)(threadIdx.x & 63u);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t yw = y0 + w * RS;    // this wave's first row
    const int64_t gx = x0 + 4 * lane;  // this lane's first column
    // rows r0 <= i < r1 of the band are rows of the grid
    const int r0 = EDGE && yw < 0 ? (int)(-yw < RS ? -yw : RS) : 0;
    const int r1 = EDGE && NY - yw < RS ? (int)(NY > yw ? NY - yw : 0) : RS;
    const int64_t origin = yw * NX + x0;
    const f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};

    f32x4 c[RS];
    const bool cols = !EDGE || (gx >= 0 && gx < NX);
    const bool cut = EDGE && !VEC && gx < NX && gx + 4 > NX;  // by the row's end: reads the row's last 16 bytes
    const int at = (int)(cut ? NX - 4 - x0 : 4 * lane);
    each_row<RS>([&](auto row) __attribute__((always_inline)) {
        constexpr int i = row;
        c[i] = z;
        if (i >= r0 && i < r1 && cols) {
            const float* p = u + (origin + i * NX) + at;
            using vec = std::conditional_t<VEC, f32x4, f32x4_a4>;
            c[i] = *reinterpret_cast<const vec*>(p);
        }
    });
    if (EDGE && !VEC && (NX & 3) && x0 + JT_W > NX)  // block-uniform
        each_row<RS>([&](auto row) __attribute__((always_inline)) {
            constexpr int i = row;
            const f32x4 e = row_end(c[i], gx + 4 - NX);
            c[i] = cut ? e : c[i];
            __builtin_amdgcn_sched_barrier(0);
        });

    bool keep[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) keep[j] = gx + j <= 0 || gx + j >= NX - 1;
    const int top = yw <= 0 && -yw < RS ? (int)-yw : -1;
    const int bottom = NY - 1 >= yw && NY - 1 - yw < RS ? (int)(NY - 1 - yw) : -1;
    jacobi_tb_sweeps<RS, WV, EDGE>(c, sweeps, w, lane, keep, top, bottom, L);

    const int hl = (int)hc / 4;
    if (lane < hl || lane >= 64 - hl || (EDGE && gx >= NX)) return;
    // the interior's rows of the band
    const int lo = (int)sweeps - w * RS, end = lo + RS * WV - 2 * (int)sweeps, hi = end < r1 ? end : r1;
    each_row<RS>([&](auto row) __attribute__((always_inline)) {
        constexpr int i = row;
        if (i >= lo && i < hi) {
            float* p = v + (origin + i * NX) + 4 * lane;
            if (VEC && NT) {
                __builtin_nontemporal_store(c[i], reinterpret_cast<f32x4*>(p));
            } else if (VEC) {
                *reinterpret_cast<f32x4*>(p) = c[i];
            } else if (!EDGE || gx + 4 <= NX) {
                *reinterpret_cast<f32x4_a4*>(p) = c[i];
            } else {
                p[0] = c[i].x;
                if (gx + 1 < NX) p[1] = c[i].y;
                if (gx + 2 < NX) p[2] = c[i].z;
            }
        }
    });
}

// Tile (bx, by) of the grid cut into tiles of 256 - 2 hc columns and
// RS * WV - 2 sweeps rows.  nx >= 4, hc is a multiple of 4, sweeps <= hc.  VEC: nx is a
// multiple of 4 and the rows are 16-byte aligned.  NT: whole-line stores that
// pass the L2 by (for grids far larger than it).  A tile below the grid reads and
// stores nothing.
template <int RS, int WV, bool VEC, bool NT>
__device__ __forceinline__ void jacobi_tb_block(const float* __restrict__ u, float* __restrict__ v, uint32_t nx,
                                                uint32_t ny, uint32_t sweeps, uint32_t hc, uint32_t bx, uint32_t by,
                                                JacobiTbLds<WV>& L) {
    const int64_t x0 = (int64_t)bx * (JT_W - 2 * hc) - hc, y0 = (int64_t)by * (RS * WV - 2 * sweeps) - sweeps;
    if (x0 <= 0 || x0 + JT_W >= (int64_t)nx || y0 <= 0 || y0 + RS * WV >= (int64_t)ny)
        jacobi_tb_region<RS, WV, VEC, NT, true>(u, v, nx, ny, sweeps, hc, x0, y0, L);
    else
        jacobi_tb_region<RS, WV, VEC, NT, false>(u, v, nx, ny, sweeps, hc, x0, y0, L);
}

}  // namespace spmd

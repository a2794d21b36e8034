// k_jacobi.hip -- JACOBI5_F32 kernel and launcher.
#include "cls_jacobi.hpp"

namespace spmd {

constexpr int JS_WAVES = 4;

// A workgroup of four waves owns 256 columns and 4 R rows.
template <int R>
__global__ __launch_bounds__(64 * JS_WAVES) void jacobi5_kernel(const float* __restrict__ u, float* __restrict__ v,
                                                                uint32_t nx, uint32_t ny, uint32_t gx) {
    const uint32_t t = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t x0 = (int64_t)(t % gx) * JS_W, y0 = ((int64_t)(t / gx) * JS_WAVES + w) * R;
    if (y0 < ny) jacobi_strip<R>(u, v, nx, ny, x0, x0 + JS_W < nx ? x0 + JS_W : nx, y0);
}

template <int R>
static void launch(const LaunchCtx& c, const float* u, float* v, uint32_t nx, uint32_t ny) {
    const uint32_t gx = (uint32_t)(((uint64_t)nx + JS_W - 1) / JS_W);
    const dim3 g = tile_grid(gx, ((uint64_t)ny + JS_WAVES * R - 1) / (JS_WAVES * R));
    dispatch((jacobi5_kernel<R>), g, dim3(64 * JS_WAVES), c.dyn_shmem, c.stream, u, v, nx, ny, gx);
}

int launch_jacobi5_f32(const LaunchCtx& c) {
    const uint32_t BX = c.block.x, BY = c.block.y;
    if (c.block.z != 1 || c.grid.z != 1) return SPMD_ERR_INVALID_DIM;
    auto u = arg<const float*>(c.args, 0);
    auto v = arg<float*>(c.args, 1);
    auto nx = arg<uint32_t>(c.args, 2);
    auto ny = arg<uint32_t>(c.args, 3);
    if (!u || !v || nx == 0 || ny == 0) return SPMD_ERR_ARGS;
    if ((uint64_t)c.grid.x * BX < nx) return SPMD_ERR_INVALID_DIM;
    const uint64_t rows = (uint64_t)c.grid.y * BY;
    const uint64_t per = (ny + rows - 1) / rows;
    const uint32_t C = next_pow2((uint32_t)per);
    if (C > 16) return SPMD_ERR_INVALID_DIM;
    const uint64_t brow = (uint64_t)BY * C;  // rows of one block row of the launch
    const bool listed = (BX == 16 && BY == 16) || (BX == 32 && BY == 8) ||
                        (BX == 64 && (BY == 1 || BY == 2 || BY == 4 || BY == 8)) ||
                        (BX == 128 && (BY == 2 || BY == 4)) || (BX == 256 && BY == 1);
    if ((brow < 4 || brow > 64) && !listed) return SPMD_ERR_INVALID_DIM;
    // The launch's blocks are fetched 256 columns at a time (coarse-grained
    // fetching along x, Section IV-A) and their rows dealt to waves; every cell
    // is computed as in its own block.  One row per wave where input and output
    // outgrow the 256 MB cache (8190 x 8191: 94 us against 101 with two), two
    // below (333 x 5000: 4.6 against 5.2; 2001 x 1999 6.6 with either).
    if ((uint64_t)nx * ny > (1ull << 25)) launch<1>(c, u, v, nx, ny);
    else launch<2>(c, u, v, nx, ny);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPMD_OK : hip_fail(e);
}

}  // namespace spmd

// k_jacobi.hip -- JACOBI5_F32 kernel and launcher.
#include "cls_jacobi.hpp"

namespace spmd {

inline __host__ __device__ uint32_t strips_of(uint32_t nx) { return (nx - 1) / JS_W + 1; }

// A workgroup of W waves owns 256 columns and R W rows.  (The strips to a row are
// counted here: as one more argument they took small launches from 4.36 to 4.57 us.)
template <int R, int W>
__global__ __launch_bounds__(64 * W) void jacobi5_kernel(const float* __restrict__ u, float* __restrict__ v,
                                                         uint32_t nx, uint32_t ny) {
    const uint32_t gx = strips_of(nx);
    const uint32_t t = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t x0 = (int64_t)(t % gx) * JS_W, y0 = ((int64_t)(t / gx) * W + w) * R;
    if (y0 < ny) jacobi_strip<R>(u, v, nx, ny, x0, x0 + JS_W < nx ? x0 + JS_W : nx, y0);
}

// The same for grids of up to 64 columns: a lane per column.
template <int R, int W>
__global__ __launch_bounds__(64 * W) void jacobi5_narrow_kernel(const float* __restrict__ u, float* __restrict__ v,
                                                                uint32_t nx, uint32_t ny) {
    const uint32_t t = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t y0 = ((int64_t)t * W + w) * R;
    if (y0 < ny) jacobi_narrow<R>(u, v, nx, ny, 0, nx, y0);
}

template <int R, int W>
static void launch(const LaunchCtx& c, const float* u, float* v, uint32_t nx, uint32_t ny) {
    const dim3 g = tile_grid(strips_of(nx), ((uint64_t)ny + W * R - 1) / (W * R));
    dispatch((jacobi5_kernel<R, W>), g, dim3(64 * W), c.dyn_shmem, c.stream, u, v, nx, ny);
}

template <int R, int W>
static void launch_narrow(const LaunchCtx& c, const float* u, float* v, uint32_t nx, uint32_t ny) {
    const dim3 g = tile_grid(1, ((uint64_t)ny + W * R - 1) / (W * R));
    dispatch((jacobi5_narrow_kernel<R, W>), g, dim3(64 * W), c.dyn_shmem, c.stream, u, v, nx, ny);
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
    // outgrow the 256 MB cache (8190 x 8191: 94 us against 101 with two), eight
    // waves to a workgroup, which share the rows between them (16384^2 352 us, 378
    // with four and 388 with sixteen; 8192^2 84.0, 85.0 and 91.7), four where rows
    // are longer (1500 x 300 000 670 against 712, 20000 x 20004 561 against 571); two
    // rows and four waves below (333 x 5000: 4.6 against 5.2; 2001 x 1999 6.6 with either).
    // Tall grids that leave many of a strip's lanes without a column take more
    // rows: up to 64 columns eight with a lane each (200 000 x 16 15.6 us, 31.1 as
    // strips of two), up to 160 four (2^18 rows of 65 40.5 against 50.2, of 100
    // 49.5 against 53.3, of 128 53.5 against 57.2; of 250 99.8 against 92.0 with
    // one).  Below 2^15 rows they take as long either way.
    const bool tall = ny >= 1u << 15;
    if (tall && nx <= 64) launch_narrow<8, 4>(c, u, v, nx, ny);
    else if (tall && nx <= 160) launch<4, 4>(c, u, v, nx, ny);
    else if ((uint64_t)nx * ny > (1ull << 25)) nx <= 1u << 14 ? launch<1, 8>(c, u, v, nx, ny) : launch<1, 4>(c, u, v, nx, ny);
    else launch<2, 4>(c, u, v, nx, ny);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPMD_OK : hip_fail(e);
}

}  // namespace spmd

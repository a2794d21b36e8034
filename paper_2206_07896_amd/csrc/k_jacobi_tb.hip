// k_jacobi_tb.hip -- JACOBI5T_F32 kernel and launcher: S fused sweeps.
#include "cls_jacobi_tb.hpp"

namespace spmd {

// Halo columns, whole groups of four.  Few sweeps of a large grid: 16, so that a
// tile's rows are whole 128-byte lines (2 sweeps of 8192^2 97 us against 104 at
// 4); with 5 or more the columns recomputed cost more (8 sweeps 112 against 107
// at 8).
__host__ __device__ inline uint32_t halo_cols(uint32_t sweeps, bool large) {
    return large && sweeps <= 4 ? 16 : (sweeps + 3) / 4 * 4;
}

// Eight words of arguments: one more took 100 sweeps of 1024^2 from 89.1 to 90.2 us.
template <int RS, int WV, bool VEC, bool NT>
__global__ __launch_bounds__(64 * WV, 4) void jacobi5_tb_kernel(const float* __restrict__ u, float* __restrict__ v,
                                                                uint32_t nx, uint32_t ny, uint32_t sweeps,
                                                                uint32_t gx) {
    __shared__ JacobiTbLds<WV> L;
    const uint32_t nt = gridDim.x * gridDim.y;
    const uint32_t tile = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, nt);
    jacobi_tb_block<RS, WV, VEC, NT>(u, v, nx, ny, sweeps, halo_cols(sweeps, NT), tile % gx, tile / gx, L);
}

namespace {

// Bands x waves of a region, by rows.
struct TbForm {
    uint32_t rs, wv;
    uint32_t rows() const { return rs * wv; }
};
constexpr TbForm kForms[] = {{6, 4}, {4, 8}, {5, 8}, {6, 8}, {8, 8}, {12, 8}};
constexpr int NFORMS = sizeof kForms / sizeof kForms[0], LARGE = NFORMS - 1;

uint64_t tiles_of(int f, uint32_t nx, uint32_t ny, uint32_t sweeps) {
    const uint64_t w = JT_W - 2 * halo_cols(sweeps, f == LARGE), h = kForms[f].rows() - 2 * sweeps;
    return (nx + w - 1) / w * ((ny + h - 1) / h);
}

// The form for a grid.  Taller regions recompute fewer halo rows but make
// fewer tiles.  96 rows where their tiles fill the chip's three resident
// blocks per CU and the grid is at least four of them high; there it is at
// least 50 MB and stores that pass the L2 by are the faster ones (8192^2 on
// buffers that no cache holds, 8 sweeps: 107 us against 115 with plain stores
// and 129 with the loads passing the L2 by).  Flat grids leave most of a
// region's rows outside: 4 sweeps of one row of 2^20 take 69 us in 96-row
// regions, 16.5 in 24; of 4 x 300 000 24.5 and 8.0; of 300 x 65 536 30.3, and 28.4
// in 48 (1000 x 16 384 within 7% either way).
// Otherwise the rows that the busiest CU works on decide: 11 sweeps of
// 1024^2 take 9.9 us at 48 rows (200 tiles), 11.7 at 40 (285), 12.2 at 32
// (515) and 11.5 at 64 (125); of 128^2, 6.5 us at 24 rows and 10.5 at 64; of
// 2048^2, 18.2 us at 64 rows, 18.5 at 48, 19.7 at 40.
int form_of(uint32_t nx, uint32_t ny, uint32_t sweeps, uint32_t cus) {
    if (ny >= 4 * kForms[LARGE].rows() && tiles_of(LARGE, nx, ny, sweeps) >= 3ull * cus) return LARGE;
    int best = 0;
    uint64_t least = ~0ull;
    for (int i = 0; i < LARGE; ++i) {
        const uint64_t rows = (tiles_of(i, nx, ny, sweeps) + cus - 1) / cus * kForms[i].rows();
        if (rows < least) {
            least = rows;
            best = i;
        }
    }
    return best;
}

template <int F, bool VEC>
void launch_form(const float* u, float* v, uint32_t nx, uint32_t ny, uint32_t sweeps, size_t dyn, hipStream_t st) {
    constexpr int RS = (int)kForms[F].rs, WV = (int)kForms[F].wv;
    const uint32_t hc = halo_cols(sweeps, F == LARGE), w = JT_W - 2 * hc, h = RS * WV - 2 * sweeps;
    const uint32_t gx = (uint32_t)(((uint64_t)nx + w - 1) / w);
    const dim3 g = tile_grid(gx, ((uint64_t)ny + h - 1) / h);
    dispatch((jacobi5_tb_kernel<RS, WV, VEC, F == LARGE>), g, dim3(64 * WV), dyn, st, u, v, nx, ny, sweeps, gx);
}

template <bool VEC>
void launch_any(int form, const float* u, float* v, uint32_t nx, uint32_t ny, uint32_t sweeps, size_t dyn,
                hipStream_t st) {
    switch (form) {
    case 0: launch_form<0, VEC>(u, v, nx, ny, sweeps, dyn, st); break;
    case 1: launch_form<1, VEC>(u, v, nx, ny, sweeps, dyn, st); break;
    case 2: launch_form<2, VEC>(u, v, nx, ny, sweeps, dyn, st); break;
    case 3: launch_form<3, VEC>(u, v, nx, ny, sweeps, dyn, st); break;
    case 4: launch_form<4, VEC>(u, v, nx, ny, sweeps, dyn, st); break;
    case 5: launch_form<5, VEC>(u, v, nx, ny, sweeps, dyn, st); break;
    }
    static_assert(NFORMS == 6, "every form has a case");
}

}  // namespace

int jacobi_tb_enqueue(const float* u, float* v, uint32_t nx, uint32_t ny, uint32_t sweeps, size_t dyn_shmem,
                      const DevInfo* dev, hipStream_t stream) {
    int form = form_of(nx, ny, sweeps, (uint32_t)dev->num_cus);
    // eight waves exchange rows through 32 KiB of LDS, four through 16
    if (dyn_shmem + 2 * sizeof(JacobiTbLds<4>) > dev->max_shmem_per_block) form = 0;
    if (nx % 4u == 0 && aligned(u, 16) && aligned(v, 16))
        launch_any<true>(form, u, v, nx, ny, sweeps, dyn_shmem, stream);
    else
        launch_any<false>(form, u, v, nx, ny, sweeps, dyn_shmem, stream);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPMD_OK : hip_fail(e);
}

int launch_jacobi5t_f32(const LaunchCtx& c) {
    // the class's grid: tiles of (256 - 2 H) x 64 cells, H = 4 or 8
    if (c.block.x != 256 || c.block.y != 1 || c.block.z != 1 || c.grid.z != 1) return SPMD_ERR_INVALID_DIM;
    auto u = arg<const float*>(c.args, 0);
    auto v = arg<float*>(c.args, 1);
    auto nx = arg<uint32_t>(c.args, 2);
    auto ny = arg<uint32_t>(c.args, 3);
    auto sweeps = arg<uint32_t>(c.args, 4);
    if (!u || !v || nx == 0 || ny == 0 || sweeps == 0 || sweeps > 8) return SPMD_ERR_ARGS;
    if (nx % 4u || !aligned(u, 16) || !aligned(v, 16)) return SPMD_ERR_ARGS;
    const uint64_t bytes = 4ull * nx * ny;
    const uintptr_t a = (uintptr_t)u, b = (uintptr_t)v;
    if (a < b + bytes && b < a + bytes) return SPMD_ERR_ARGS;  // u and v overlap
    const uint64_t halo = sweeps <= 4 ? 4 : 8;
    if (c.grid.x * (JT_W - 2 * halo) < nx || c.grid.y * 64ull < ny) return SPMD_ERR_INVALID_DIM;
    return jacobi_tb_enqueue(u, v, nx, ny, sweeps, c.dyn_shmem, c.dev, c.stream);
}

}  // namespace spmd

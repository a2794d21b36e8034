// k_gemm.hip -- GEMM_F32 kernels and launcher.
#include <iterator>

#include "cls_gemm.hpp"
#include "cls_jacobi.hpp"  // xcd_tile

namespace spmd {

// Direct-to-LDS form: NS slices in flight (4 at tiles 64 and 128; 3 at
// tile 256, whose stages are twice as large).
template <int T, int NS, int V>
__global__ __launch_bounds__(256) void gemm_f32_dma_kernel(const float* __restrict__ A, const float* __restrict__ B,
                                                            float* __restrict__ C, uint32_t M, uint32_t N, uint32_t K,
                                                            uint32_t gx) {
    constexpr int SZ = 2 * T * GEMM_DMA_KT;
    __shared__ __attribute__((aligned(16))) float S0[SZ];
    __shared__ __attribute__((aligned(16))) float S1[SZ];
    __shared__ __attribute__((aligned(16))) float S2[NS > 2 ? SZ : 4];
    __shared__ __attribute__((aligned(16))) float S3[NS > 3 ? SZ : 4];
    gemm_block_dma<T, NS, V>(A, B, C, M, N, K, blockIdx.x % gx, blockIdx.x / gx, S0, S1, S2, S3);
}

template <int RT, int W, int D, typename Off>
__global__ __launch_bounds__(64 * W) void gemm_f32_ksplit_kernel(const float* __restrict__ A,
                                                                 const float* __restrict__ B, float* __restrict__ C,
                                                                 uint32_t M, uint32_t N, uint32_t K, uint32_t gx,
                                                                 uint32_t tiles) {
    __shared__ GemmKsplitLds<RT, W> L;
    for (uint32_t id = blockIdx.x; id < tiles; id += gridDim.x) {
        const uint32_t t = xcd_tile(id, tiles);  // a range of tiles per XCD: their rows of A meet in its L2
        gemm_block_ksplit<RT, W, D, Off>(A, B, C, M, N, K, t % gx, t / gx, L);
        __syncthreads();  // the next tile reuses the LDS
    }
}

namespace {

// The forms, and what one tile takes on a CU, in 0.1 ns: per unit of K, and
// beside it for its start and the way out of C.  Per K measured at shapes that
// fill the 256 CUs with one or more tiles: 4096^3, 2048^3, 3000^3 and 1536^3 with
// 16-byte rows; 4095^3, 2047 x 2049 x 2047 and 3001 x 2999 x 3001 without; 512 x
// 512 x 4096 and 1023 x 1025 x 1027 for the 32 x 32 tiles.  Beside it fitted to
// 242 shapes of K from 1 to 512: the larger the tile, the nearer it runs to the
// matrix cores' rate, the more a shape that does not fill a round of tiles
// leaves idle, and the longer its C takes with no other block's products beside
// it (8192 x 8192 x 16: 52 us on 64 x 64 tiles, 57 on 128 x 128, 64 on 256 x 256;
// 4096 x 4096 x 256 75 on all three).  Without 16-byte rows 64 x 64 tiles by 4-byte
// loads take short K (2047 x 2049 x 64: 12.2 us, 18.3 split over waves).
enum class GemmForm { SPLIT32, SPLIT64, DMA64, DMA128, DMA256 };
struct GemmCost {
    GemmForm form;
    uint32_t tile, per_k, beside;
    size_t lds;  // of a block
};
constexpr size_t dma_lds(size_t tile, size_t stages) { return 8 * tile * GEMM_DMA_KT * stages + 16 * (4 - stages); }
constexpr GemmCost GEMM_ALIGNED[] = {{GemmForm::DMA256, 256, 2620, 160000, dma_lds(256, 3)},
                                     {GemmForm::DMA128, 128, 690, 30000, dma_lds(128, 4)},
                                     {GemmForm::DMA64, 64, 194, 4000, dma_lds(64, 4)},
                                     {GemmForm::SPLIT32, 32, 75, 4000, 0}};
constexpr GemmCost GEMM_ANY[] = {{GemmForm::DMA256, 256, 2890, 160000, dma_lds(256, 3)},
                                 {GemmForm::DMA128, 128, 770, 40000, dma_lds(128, 4)},
                                 {GemmForm::SPLIT64, 64, 224, 6000, sizeof(GemmKsplitLds<2, 4>)},
                                 {GemmForm::DMA64, 64, 240, 1000, dma_lds(64, 4)},
                                 {GemmForm::SPLIT32, 32, 80, 1000, 0}};
// Of 16-byte rows that don't begin on 128-byte lines (N % 32), a 64-column piece
// ends in two lines that others write too: 10000 x 10000 x 16 94 us on 128 x 128
// tiles, 112 on 64 x 64.
constexpr uint32_t GEMM_CUT_LINES = 4000;

uint64_t tiles_of(uint32_t M, uint32_t N, uint32_t t) {
    return (((uint64_t)M + t - 1) / t) * (((uint64_t)N + t - 1) / t);
}

// A launch's grid says which tiles its blocks own, but not on how many CUs
// they run: the form is chosen by the shape alone, the least (rounds of tiles
// over the CUs) x (time of a tile).  1000 x 901 x 1111 at the 128 x 128 tiles of
// its launch kept 64 CUs busy for 174 us (64 x 64 split: 25.4 us); 4096^3 at 64 x 64
// tiles took 1059 us (256 x 256: 958 us).  Ties go to the larger tile.  Forms
// whose offsets (32 bits) or grid (32 bits of threads) a shape exceeds, or whose
// LDS is more than the launch's dynamic shared memory leaves (`room`), are left
// out; the 32 x 32 split form has a 64-bit build, strides over its tiles and
// takes four waves where eight don't fit.
GemmForm gemm_form(uint32_t M, uint32_t N, uint32_t K, bool vec, int num_cus, size_t room) {
    GemmForm best = GemmForm::SPLIT32;
    uint64_t least = ~0ull;
    const GemmCost* const first = vec ? GEMM_ALIGNED : GEMM_ANY;
    const GemmCost* const last = vec ? std::end(GEMM_ALIGNED) : std::end(GEMM_ANY);
    for (const GemmCost* p = first; p != last; ++p) {
        const GemmCost& f = *p;
        const uint64_t tiles = tiles_of(M, N, f.tile);
        if (f.form != GemmForm::SPLIT32) {
            if (4ull * f.tile * K >= (1ull << 31) || 4ull * GEMM_DMA_KT * N >= (1ull << 31)) continue;
            if (tiles >= (1ull << 24) || f.lds > room) continue;
        }
        const uint64_t cut = vec && f.form == GemmForm::DMA64 && N % 32 ? GEMM_CUT_LINES : 0;
        const uint64_t c = (tiles + num_cus - 1) / num_cus * ((uint64_t)f.per_k * K + f.beside + cut);
        if (c < least) {
            least = c;
            best = f.form;
        }
    }
    return best;
}

}  // namespace

int launch_gemm_f32(const LaunchCtx& c) {
    if (c.block.x != 256 || c.block.y != 1 || c.block.z != 1 || c.grid.z != 1) return SPMD_ERR_INVALID_DIM;
    auto A = arg<const float*>(c.args, 0);
    auto B = arg<const float*>(c.args, 1);
    auto C = arg<float*>(c.args, 2);
    auto M = arg<uint32_t>(c.args, 3);
    auto N = arg<uint32_t>(c.args, 4);
    auto K = arg<uint32_t>(c.args, 5);
    if (!A || !B || !C || M == 0 || N == 0 || K == 0) return SPMD_ERR_ARGS;
    uint32_t T = 0;  // the launch's tile
    for (uint32_t t : {256u, 128u, 64u})
        if ((uint64_t)c.grid.x * t >= N && (uint64_t)c.grid.y * t >= M) T = t;
    if (!T) return SPMD_ERR_INVALID_DIM;
    const bool vec = aligned(A, 16) && K % 4 == 0 && aligned(B, 16) && N % 4 == 0;
    // What the launch reserves has to fit beside its own tile's stages: four of
    // 16 deep (three at 256), rows off 16 bytes two, each row padded by 4 floats.
    const bool dma_rows = vec && (uint64_t)T * K < (1ull << 31) && (uint64_t)GEMM_DMA_KT * N < (1ull << 31);
    const size_t own = dma_rows ? dma_lds(T, T == 256 ? 3 : 4) : 16 * GEMM_DMA_KT * ((size_t)T + 4);
    if (own + c.dyn_shmem > c.dev->max_shmem_per_block) return SPMD_ERR_SHMEM;
    const size_t dyn = c.dyn_shmem, room = c.dev->max_shmem_per_block - dyn;
    const hipStream_t s = c.stream;
    auto dma = [&](auto kernel, uint32_t t) {
        dispatch(kernel, dim3((uint32_t)tiles_of(M, N, t)), dim3(256), (uint32_t)dyn, s, A, B, C, M, N, K,
                 (N + t - 1) / t);
    };
    auto split = [&](auto kernel, uint32_t t, uint32_t threads) {
        const uint64_t tiles = tiles_of(M, N, t);
        dispatch(kernel, dim3((uint32_t)(tiles < (1u << 22) ? tiles : (1u << 22))), dim3(threads), (uint32_t)dyn, s, A,
                 B, C, M, N, K, (uint32_t)(((uint64_t)N + t - 1) / t), (uint32_t)tiles);
    };
    switch (gemm_form(M, N, K, vec, c.dev->num_cus, room)) {
    case GemmForm::DMA256:
        if (vec) dma(gemm_f32_dma_kernel<256, 3, 4>, 256);
        else dma(gemm_f32_dma_kernel<256, 3, 1>, 256);
        break;
    case GemmForm::DMA128:
        if (vec) dma(gemm_f32_dma_kernel<128, 4, 4>, 128);
        else dma(gemm_f32_dma_kernel<128, 4, 1>, 128);
        break;
    case GemmForm::DMA64:
        if (vec) dma(gemm_f32_dma_kernel<64, 4, 4>, 64);
        else dma(gemm_f32_dma_kernel<64, 4, 1>, 64);
        break;
    case GemmForm::SPLIT64: split(gemm_f32_ksplit_kernel<2, 4, 4, uint32_t>, 64, 256); break;
    case GemmForm::SPLIT32:
        static_assert(sizeof(GemmKsplitLds<1, 4>) <= 16 * GEMM_DMA_KT * (64 + 4), "fits wherever the least tile does");
        if (sizeof(GemmKsplitLds<1, 8>) > room)
            split(gemm_f32_ksplit_kernel<1, 4, 2, uint64_t>, 32, 256);
        else if (4ull * 32 * K < (1ull << 31) && 4ull * 8 * N < (1ull << 31))
            split(gemm_f32_ksplit_kernel<1, 8, 2, uint32_t>, 32, 512);
        else
            split(gemm_f32_ksplit_kernel<1, 8, 2, uint64_t>, 32, 512);
        break;
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPMD_OK : hip_fail(e);
}

}  // namespace spmd

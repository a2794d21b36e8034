// k_hist.hip -- HIST256_U32 kernels and launcher.  The launch enqueues a
// clear of the 256 output bins (a fill kernel, so the pair can be captured
// into a graph) and then the counting grid; for few keys one block that writes
// them.
#include <algorithm>

#include "cls_hist.hpp"

namespace spmd {

__global__ __launch_bounds__(256) void hist_clear_kernel(uint32_t* hist) { hist[threadIdx.x] = 0u; }

constexpr int HIST_THREADS = 1024;

// The launch's shape: a block of its size per segment.
template <int B>
__global__ __launch_bounds__(B) void hist256_kernel(const uint32_t* __restrict__ keys, uint32_t* hist, uint32_t n,
                                                     uint32_t seg) {
    __shared__ HistLds<HIST_COPIES> L;
    const uint64_t lo = (uint64_t)blockIdx.x * seg;
    const uint64_t hi = lo + seg < (uint64_t)n ? lo + seg : (uint64_t)n;
    hist_block<B, HIST_COPIES>(keys, hist, lo, hi, L);
}

__global__ __launch_bounds__(HIST_THREADS) void hist256_alone_kernel(const uint32_t* __restrict__ keys, uint32_t* hist,
                                                                      uint32_t n) {
    __shared__ HistLds<HIST_COPIES> L;
    hist_block<HIST_THREADS, HIST_COPIES, true>(keys, hist, 0, n, L);
}

// Blocks (of 1024 threads) for n keys on the device's CUs; 0: one block alone,
// without the clear.  (Not for a launch with dynamic shared memory, here as for
// scans and compactions: what it reserves bounds how many of its own blocks a CU
// takes, and would mean something else in others.)  The counts do not depend on the launch's grid, but every
// block adds up to 256 bins to the same 1 KiB, 18 billion a second in all:
// launched in 1024 blocks 2^16 keys took 22 us, 2^20 23, 2^24 27 to 31; in 64
// blocks of 256 2^24 65, 2^26 252.  Fewer blocks read more slowly.  The fastest,
// with those beside it, in us: 2^16 keys 4.1 in 16 (4.4 in 8, 4.7 in 64), 2^17 4.3
// in 32, 2^18 4.9 and 2^20 6.5 in 64 (32: 5.1 and 7.9; 128: 6.0 and 6.8), 2^22
// 9.6 in 128 (64: 12.2, 256: 10.5), 2^23 11.8 in 192 (128: 13.3, 256: 12.5), from
// 2^24 on 17.4 in 256, a block per CU.  Up to 2^13 one block's time is less than
// the clear's.
static uint32_t hist_blocks(uint32_t n, uint32_t cus) {
    if (n <= 1u << 13) return 0;
    const uint32_t g = n < 1u << 17   ? cus / 16
                       : n < 1u << 18 ? cus / 8
                       : n < 1u << 21 ? cus / 4
                       : n < 1u << 23 ? cus / 2
                       : n < 1u << 24 ? cus / 4 * 3
                                      : cus;
    return std::max(g, 1u);
}

uint32_t hist_launches(uint32_t n) { return hist_blocks(n, 256) ? 2u : 1u; }

int launch_hist256_u32(const LaunchCtx& c) {
    const uint32_t B = c.block.x;
    if (c.block.y != 1 || c.block.z != 1 || c.grid.y != 1 || c.grid.z != 1) return SPMD_ERR_INVALID_DIM;
    if (!is_pow2(B) || B < 64 || B > 1024) return SPMD_ERR_INVALID_DIM;
    auto keys = arg<const uint32_t*>(c.args, 0);
    auto hist = arg<uint32_t*>(c.args, 1);
    auto n = arg<uint32_t>(c.args, 2);
    if ((!keys && n) || !hist) return SPMD_ERR_ARGS;
    const uint32_t G = c.grid.x;
    const uint64_t seg64 = segment_len(n, G);
    if (seg64 > 0xFFFFFFFFull) return SPMD_ERR_INVALID_DIM;
    const uint32_t blocks = hist_blocks(n, (uint32_t)c.dev->num_cus);
    if (n && c.dyn_shmem == 0 && blocks == 0) {
        dispatch(hist256_alone_kernel, dim3(1), dim3(HIST_THREADS), 0, c.stream, keys, hist, n);
    } else {
        dispatch(hist_clear_kernel, dim3(1), dim3(256), 0, c.stream, hist);
        if (n && c.dyn_shmem == 0) {
            const uint32_t seg = (uint32_t)segment_len(n, blocks);
            dispatch(hist256_kernel<HIST_THREADS>, dim3(blocks), dim3(HIST_THREADS), 0, c.stream, keys, hist, n, seg);
        } else if (n) {
            const dim3 g(G), b(B);
            const uint32_t seg = (uint32_t)seg64;
            switch (B) {
            case 64: dispatch(hist256_kernel<64>, g, b, c.dyn_shmem, c.stream, keys, hist, n, seg); break;
            case 128: dispatch(hist256_kernel<128>, g, b, c.dyn_shmem, c.stream, keys, hist, n, seg); break;
            case 256: dispatch(hist256_kernel<256>, g, b, c.dyn_shmem, c.stream, keys, hist, n, seg); break;
            case 512: dispatch(hist256_kernel<512>, g, b, c.dyn_shmem, c.stream, keys, hist, n, seg); break;
            case 1024: dispatch(hist256_kernel<1024>, g, b, c.dyn_shmem, c.stream, keys, hist, n, seg); break;
            }
        }
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPMD_OK : hip_fail(e);
}

}  // namespace spmd

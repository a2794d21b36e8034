// k_reduce.hip -- REDUCE_I32 kernel and launcher.
//
// Workspace: the two-level completion ticket and the launch epoch
// (REDUCE_CTL_BYTES, counters on separate cache lines), then one u64 status
// word per block (per workgroup in the persistent form, which needs fewer),
// tagged with the epoch: the finishing block re-arms the ticket and
// advances the epoch, so the next launch needs no clearing.
#include <algorithm>

#include "cls_reduce.hpp"
#include "common.hpp"

namespace spmd {

constexpr size_t REDUCE_WS_HEADER = REDUCE_CTL_BYTES;

template <int B>
__global__ __launch_bounds__(B) void reduce_i32_kernel(const int32_t* __restrict__ x, int32_t* partials,
                                                        int32_t* out, uint32_t n, uint32_t seg, uint32_t* ws,
                                                        uint32_t* err) {
    __shared__ ReduceLds<B> L;
    uint64_t* status = reinterpret_cast<uint64_t*>(reinterpret_cast<uint8_t*>(ws) + REDUCE_WS_HEADER);
    reduce_block<B>(x, partials, out, n, seg, gridDim.x, blockIdx.x, ws, status, err, L);
}

// The persistent form: workgroup w runs logical blocks [K w, K w + K).
template <int B, int K>
__global__ __launch_bounds__(B) void reduce_i32_pkernel(const int32_t* __restrict__ x, int32_t* partials,
                                                         int32_t* out, uint32_t n, uint32_t seg, uint32_t G,
                                                         uint32_t* ws, uint32_t* err) {
    __shared__ ReduceLds<B> L;
    __shared__ uint32_t wsum[K][B / 64];
    uint64_t* status = reinterpret_cast<uint64_t*>(reinterpret_cast<uint8_t*>(ws) + REDUCE_WS_HEADER);
    reduce_blocks<B, K>(x, partials, out, n, seg, G, gridDim.x, blockIdx.x, ws, status, err, L, wsum);
}

// Short segments: a wave per logical block.
template <int J>
__global__ __launch_bounds__(256) void reduce_i32_wkernel(const int32_t* __restrict__ x, int32_t* partials,
                                                          int32_t* out, uint32_t n, uint32_t seg, uint32_t G,
                                                          uint32_t* ws, uint32_t* err) {
    __shared__ ReduceLds<256> L;
    uint64_t* status = reinterpret_cast<uint64_t*>(reinterpret_cast<uint8_t*>(ws) + REDUCE_WS_HEADER);
    reduce_waves<J>(x, partials, out, n, seg, G, gridDim.x, blockIdx.x, ws, status, err, L);
}

size_t ws_reduce_i32(spmd_dim3 grid, spmd_dim3, uint64_t) { return REDUCE_WS_HEADER + 8ull * grid.x; }

// Logical blocks per workgroup: the largest K in {1, 2, 4, 8} that still
// leaves at least one workgroup per resident slot (2 for 4096 blocks of 256:
// 2048 workgroups of 256 threads fill the device).  At K = 1 the
// one-block-per-workgroup kernel runs.  More than 256 threads run fewer than 16
// blocks to a CU (launch_reduce_i32), so K stays below 16 / (2048 / B) there.
template <int B>
constexpr uint32_t REDUCE_K_MAX = B > 256 ? B / 256 : 8;

template <int B>
static uint32_t reduce_blocks_per_wg(uint32_t G, int num_cus) {
    static const int per_cu = [] {  // one query per block size (one GPU architecture)
        int v = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, reduce_i32_pkernel<B, 2>, B, 0) != hipSuccess) v = 0;
        return v;
    }();
    if (per_cu < 1) return 1;
    const uint64_t slots = (uint64_t)per_cu * (uint64_t)num_cus;
    uint32_t K = 1;
    while (K < REDUCE_K_MAX<B> && (uint64_t)G >= 2ull * K * slots) K *= 2;
    return K;
}

template <int B>
static void launch_reduce_b(uint32_t G, size_t dyn, hipStream_t s, const int32_t* x, int32_t* partials,
                            int32_t* out, uint32_t n, uint32_t seg, uint32_t* ws, uint32_t* err,
                            int num_cus) {
    const uint32_t K = reduce_blocks_per_wg<B>(G, num_cus);
    const dim3 b(B);
    switch (K) {
    case 1: dispatch(reduce_i32_kernel<B>, dim3(G), b, dyn, s, x, partials, out, n, seg, ws, err); break;
    case 2: dispatch((reduce_i32_pkernel<B, 2>), dim3((G + 1) / 2), b, dyn, s, x, partials, out, n, seg, G, ws, err); break;
    case 4:
        if constexpr (REDUCE_K_MAX<B> >= 4)
            dispatch((reduce_i32_pkernel<B, 4>), dim3((G + 3) / 4), b, dyn, s, x, partials, out, n, seg, G, ws, err);
        break;
    case 8:
        if constexpr (REDUCE_K_MAX<B> >= 8)
            dispatch((reduce_i32_pkernel<B, 8>), dim3((G + 7) / 8), b, dyn, s, x, partials, out, n, seg, G, ws, err);
        break;
    }
}

// Logical blocks in flight per wave where a wave takes them (0: a workgroup
// does).  A block's own threads have nothing to do where its segment is short:
// 2^20 elements in 4096 blocks of 256 threads are 64 loads of 16 bytes a block,
// 6.4 us, 4.8 with a wave each; 2^22 in 4096 blocks of 1024 32.6 and 5.6, 2^24 in
// 16 384 of 512 42.8 and 11.0, 2^26 in 65 536 of 256 70.4 and 48.4.  From 4096
// elements on a block is as fast (2^24 in 4096 of 256: 14.5 us both ways), then
// faster (2^26: 46.2 against 52.8), with few blocks sooner (2^20 in 256 of 1024:
// 6.0 against 6.75, 2^18 in 256 of 128: 5.5 against 5.1).  Two blocks to a wave
// where that leaves two workgroups to a CU (4096 blocks 5.6 us against 5.7 with
// one, 16 384 9.0 against 9.8, but 2048 5.15 against 5.0).
static uint32_t wave_blocks(uint32_t seg, uint32_t G, int cus) {
    if (seg > (G >= 4u * (uint32_t)cus ? 2048u : 1024u)) return 0;
    return G >= 16u * (uint32_t)cus ? 2 : 1;
}

int launch_reduce_i32(const LaunchCtx& c) {
    const uint32_t B = c.block.x;
    if (c.block.y != 1 || c.block.z != 1 || c.grid.y != 1 || c.grid.z != 1) return SPMD_ERR_INVALID_DIM;
    if (!is_pow2(B) || B < 64 || B > 1024) return SPMD_ERR_INVALID_DIM;
    auto x = arg<const int32_t*>(c.args, 0);
    auto partials = arg<int32_t*>(c.args, 1);
    auto out = arg<int32_t*>(c.args, 2);
    auto n = arg<uint32_t>(c.args, 3);
    auto ws = arg<uint32_t*>(c.args, 4);
    if ((!x && n) || !partials || !out) return SPMD_ERR_ARGS;
    if (!ws || !aligned(ws, 16)) return SPMD_ERR_WORKSPACE;
    const uint32_t G = c.grid.x;
    const uint64_t seg64 = segment_len(n, G);
    if (seg64 > 0xFFFFFFFFull) return SPMD_ERR_INVALID_DIM;
    const uint32_t seg = (uint32_t)seg64;
    uint32_t* err = c.dev->err_word;
    const int cus = c.dev->num_cus;
    // (four waves' LDS is a few bytes more than a small block's own)
    const bool room = c.dyn_shmem + sizeof(ReduceLds<256>) <= c.dev->max_shmem_per_block;
    if (const uint32_t J = room ? wave_blocks(seg, G, cus) : 0) {
        const dim3 g((G + 4 * J - 1) / (4 * J)), b(256);
        if (J == 2) dispatch((reduce_i32_wkernel<2>), g, b, c.dyn_shmem, c.stream, x, partials, out, n, seg, G, ws, err);
        else dispatch((reduce_i32_wkernel<1>), g, b, c.dyn_shmem, c.stream, x, partials, out, n, seg, G, ws, err);
        hipError_t e = hipGetLastError();
        return e == hipSuccess ? SPMD_OK : hip_fail(e);
    }
    // Sixteen blocks to a CU are enough waves at 256 threads each; more threads
    // only share the same loads (2^26 in 4096 blocks of 1024: 44.6 us on 256 threads
    // each, 114 on their own).
    switch (G >= 16u * (uint32_t)cus ? std::min(B, 256u) : B) {
    case 64: launch_reduce_b<64>(G, c.dyn_shmem, c.stream, x, partials, out, n, seg, ws, err, cus); break;
    case 128: launch_reduce_b<128>(G, c.dyn_shmem, c.stream, x, partials, out, n, seg, ws, err, cus); break;
    case 256: launch_reduce_b<256>(G, c.dyn_shmem, c.stream, x, partials, out, n, seg, ws, err, cus); break;
    case 512: launch_reduce_b<512>(G, c.dyn_shmem, c.stream, x, partials, out, n, seg, ws, err, cus); break;
    case 1024: launch_reduce_b<1024>(G, c.dyn_shmem, c.stream, x, partials, out, n, seg, ws, err, cus); break;
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPMD_OK : hip_fail(e);
}

}  // namespace spmd

// mlp.hip -- kernels of the schedule cost model (spmd_mlp.h).
//
// The layers are contractions and run on the matrix cores in fp32
// (v_mfma_f32_32x32x2f32).  That instruction is, bit for bit, the chain
// fma(a1, b1, fma(a0, b0, c)) -- subnormals, infinities and NaN included --
// so a layer accumulated over k = 0, 1, 2, ... rounds exactly as one FMA
// after another would.
//
// Forward and choose hold the activations transposed (units down the rows of
// the matrix product, model rows across its columns), so a layer's result is
// the next layer's operand where it lies, with no exchange between lanes:
// accumulator register r holds, in lanes 0-31 and 32-63, two units of the
// model row lane % 32, and a k step of the next layer wants exactly two k per
// column, one per half-wave.  The weights' rows are permuted (unit_of) so that
// those two units are 2r and 2r + 1, i.e. k runs in its natural order.
//
// Backward contracts over the model rows instead; a chunk of rows goes through
// LDS, where it is read with rows across lanes (the error's way back) and with
// units across lanes (the weight gradients).
//
// Nothing depends on scheduling: every sum runs in a fixed order, so
// gradients are reproducible.
#include <algorithm>

#include "common.hpp"
#include "spmd_mlp.h"
#include "warp32.hpp"

namespace spmd {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // any float's address

constexpr int DIN = SPMD_MLP_DIN, HID = SPMD_MLP_H, NP = SPMD_MLP_NPARAM;
constexpr int OFF_W1 = 0, OFF_B1 = DIN * HID, OFF_W2 = OFF_B1 + HID, OFF_B2 = OFF_W2 + HID * HID,
              OFF_W3 = OFF_B2 + HID, OFF_B3 = OFF_W3 + HID;
static_assert(OFF_B3 + 1 == NP, "parameter layout");
static_assert(DIN == 12 && HID == 64, "the operand layouts below");
constexpr int MLP_ROWS = 64;  // rows per partial sum that a workspace holds; none has fewer

__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Accumulator register r of half-wave h is matrix row 8*(r/4) + 4*h + r%4.
__device__ __forceinline__ int acc_row(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }
// The unit at matrix row m of a 32-row tile: register r holds units 2r, 2r+1.
__device__ __forceinline__ int unit_of(int m) { return 2 * (4 * (m >> 3) + (m & 3)) + ((m >> 2) & 1); }

// One model's weights as matrix operands.
struct MlpWeights {
    alignas(16) float a1[2][DIN / 4][64][2];   // [unit tile][k step / 2][lane][k step % 2]
    alignas(16) float a2[2][HID / 8][64][4];   // [unit tile][k step / 4][lane][k step % 4]
    alignas(16) float b1[2][2][16];            // [unit tile][half-wave][register]
    alignas(16) float b2[2][2][16];
    alignas(16) float w3[HID];
    float b3;
};

// max(v, 0), NaN to 0, for v out of arithmetic: the middle of v, 0 and infinity
// is one instruction, where fmaxf first quietens v (and the compiler makes an
// fmaxf of it as soon as it sees the infinity).
__device__ __forceinline__ float relu(float v) {
    float inf;
    asm("s_mov_b32 %0, 0x7f800000" : "=s"(inf));
    return __builtin_amdgcn_fmed3f(v, 0.0f, inf);
}

// By T threads; every load is issued before the first is waited for (a round
// trip a weight, 19 of them, was a third of the forward pass).
template <int T>
__device__ __forceinline__ void stage_weights(MlpWeights& S, const float* __restrict__ params) {
    static_assert(HID * HID % T == 0, "whole rounds");
    constexpr int N1 = (DIN * HID + T - 1) / T, N2 = HID * HID / T;
    float* a1 = &S.a1[0][0][0][0];
    float* a2 = &S.a2[0][0][0][0];
    const int tid = threadIdx.x;
    float v1[N1], v2[N2], vb[3] = {};
#pragma unroll
    for (int p = 0; p < N1; ++p) {
        const int i = tid + p * T < DIN * HID ? tid + p * T : 0;
        const int e = i & 1, lane = (i >> 1) & 63, q = (i >> 7) % (DIN / 4), t = i / (DIN / 4 * 128);
        v1[p] = params[OFF_W1 + (2 * (2 * q + e) + (lane >> 5)) * HID + 32 * t + unit_of(lane & 31)];
    }
#pragma unroll
    for (int p = 0; p < N2; ++p) {
        const int i = tid + p * T;
        const int e = i & 3, lane = (i >> 2) & 63, q = (i >> 8) & 7, t = i >> 11;
        v2[p] = params[OFF_W2 + (2 * (4 * q + e) + (lane >> 5)) * HID + 32 * t + unit_of(lane & 31)];
    }
    const int r = tid & 15, h = (tid >> 4) & 1, t = (tid >> 5) & 1;
    if (tid < HID) {
        vb[0] = params[OFF_B1 + 32 * t + 2 * r + h];
        vb[1] = params[OFF_B2 + 32 * t + 2 * r + h];
        vb[2] = params[OFF_W3 + tid];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < N1; ++p)
        if (tid + p * T < DIN * HID) a1[tid + p * T] = v1[p];
#pragma unroll
    for (int p = 0; p < N2; ++p) a2[tid + p * T] = v2[p];
    if (tid < HID) {
        S.b1[t][h][r] = vb[0];
        S.b2[t][h][r] = vb[1];
        S.w3[tid] = vb[2];
        if (tid == 0) S.b3 = params[OFF_B3];
    }
}

__device__ __forceinline__ f32x16 load_bias(const float* p) {
    f32x16 v;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 b = *reinterpret_cast<const f32x4*>(p + 4 * q);
        v[4 * q] = b.x;
        v[4 * q + 1] = b.y;
        v[4 * q + 2] = b.z;
        v[4 * q + 3] = b.w;
    }
    return v;
}

// What the second layer starts from: its biases and its first weights.
template <int RT>
struct Upper {
    f32x16 h2[2][RT];
    f32x4 a[2];
    __device__ __forceinline__ void load(const MlpWeights& S) {
        const int lane = (int)lane64(), half = lane >> 5;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            a[t] = *reinterpret_cast<const f32x4*>(S.a2[t][0][lane]);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) h2[t][rt] = load_bias(S.b2[t][half]);
        }
    }
};

// Layers after the first for 32 RT model rows of one wave: U loaded, h1[t][rt]
// the first layer's sums (unit tile, row tile; used up), b3 the last layer's
// bias.  Returns the prediction of row `lane` (RT 1: of row lane % 32).  With
// STORE, the hidden activations go to h1t/h2t (feature-major), rows row0 + 0..63
// below n.  Weights are read from LDS one step of four k ahead of the 8 RT matrix
// steps that they serve (the sched_barriers keep them there: left to itself, the
// compiler read each right before its use and both waves of a SIMD waited);
// `then` runs when h1 is free, before the last layer, which needs no matrix step.
template <bool STORE, int RT, typename Then>
__device__ __forceinline__ float upper_layers(const MlpWeights& S, float b3, f32x16 (&h1)[2][RT], Upper<RT>& U,
                                              uint32_t row0, uint32_t n, float* h1t, float* h2t, Then then) {
#pragma clang fp contract(fast)
    const int lane = (int)lane64(), half = lane >> 5;
    f32x4 w3[HID / 4];
#pragma unroll
    for (int q = 0; q < HID / 8; ++q) {
        f32x4 next[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) next[t] = *reinterpret_cast<const f32x4*>(S.a2[t][q < 7 ? q + 1 : q][lane]);
        if (q == HID / 8 - 1) {
#pragma unroll
            for (int j = 0; j < HID / 4; ++j) w3[j] = *reinterpret_cast<const f32x4*>(S.w3 + 4 * j);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int s = 4 * q + e;  // units 2s and 2s + 1 of the first layer
            float v[RT];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                v[rt] = relu(h1[s >> 4][rt][s & 15]);
                if (STORE) {
                    const uint32_t i = row0 + 32u * rt + (lane & 31);
                    if (i < n) h1t[(uint64_t)(2 * s + half) * n + i] = v[rt];
                }
            }
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) U.h2[t][rt] = mfma32(U.a[t][e], v[rt], U.h2[t][rt]);
        }
        U.a[0] = next[0];
        U.a[1] = next[1];
        __builtin_amdgcn_sched_barrier(0);
    }
    then();
    float y = b3;
#pragma unroll
    for (int t = 0; t < 2; ++t)
        // Exchanging halves puts one unit of all rows into a register
        // (row = lane), and the last layer's sum runs over the units in order.
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float v0 = relu(U.h2[t][0][r]), v1 = relu(U.h2[t][RT - 1][r]);
            const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(v0), __float_as_uint(v1), false, false);
            const float u0 = __uint_as_float(sw[0]), u1 = __uint_as_float(sw[1]);
            const int j = 32 * t + 2 * r;
            if (STORE && RT == 1) {
                const uint32_t i = row0 + (lane & 31);
                if (i < n) h2t[(uint64_t)(j + half) * n + i] = v0;
            } else if (STORE) {
                const uint32_t i = row0 + lane;
                if (i < n) {
                    h2t[(uint64_t)j * n + i] = u0;
                    h2t[(uint64_t)(j + 1) * n + i] = u1;
                }
            }
            y += u0 * w3[j / 4][j % 4];
            y += u1 * w3[j / 4][j % 4 + 1];
        }
    return y;
}

// The first layer's k steps 2 Q0 .. 5 on top of h1, a[t][q - Q0] their weights;
// x[rt][s] is normalised input 4 Q0 + 2s + lane/32 of row 32 rt + lane%32.
template <int Q0, int RT>
__device__ __forceinline__ void first_layer(const f32x2 (&a)[2][DIN / 4 - Q0], const float (&x)[RT][DIN / 2 - 2 * Q0],
                                            f32x16 (&h1)[2][RT]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = Q0; q < DIN / 4; ++q)
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) h1[t][rt] = mfma32(a[t][q - Q0][e], x[rt][2 * (q - Q0) + e], h1[t][rt]);
}
template <int Q0>
__device__ __forceinline__ void first_weights(const MlpWeights& S, f32x2 (&a)[2][DIN / 4 - Q0]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int q = Q0; q < DIN / 4; ++q) a[t][q - Q0] = *reinterpret_cast<const f32x2*>(S.a1[t][q][lane64()]);
}

constexpr int FW_THREADS = 512, FW_ROWS = 32;

// A wave per 32 rows, eight to a block.  STORE: also the activations.  Bound by
// the matrix cores (152 of their 64-cycle steps per 64 rows, 4 us) behind the
// start of the launch, the staging of the weights and the stores: 60 000 rows with
// stores 15 to 17 us, against 20.1 with 64 rows to a wave (one wave per SIMD, the
// inputs' round trip after the weights') and 49.8 with a thread per row on the
// vector unit.
template <bool STORE>
__global__ __launch_bounds__(FW_THREADS) void mlp_forward_kernel(const float* __restrict__ params,
                                                                 const float* __restrict__ norm,
                                                                 const float* __restrict__ x, uint32_t n,
                                                                 float* __restrict__ y, float* h1t, float* h2t) {
    __shared__ MlpWeights S;
    const int lane = (int)lane64(), half = lane >> 5;
    const uint32_t row0 = (blockIdx.x * (FW_THREADS / 64) + (threadIdx.x >> 6)) * FW_ROWS;
    const uint32_t row = row0 + (lane & 31);
    const float* xr = x + (uint64_t)(row < n ? row : n - 1) * DIN;  // past the end: the last row, not stored
    float xn[1][DIN / 2], mu[DIN / 2], sd[DIN / 2];
#pragma unroll
    for (int s = 0; s < DIN / 2; ++s) {
        xn[0][s] = xr[2 * s + half];
        mu[s] = norm[2 * s + half];
        sd[s] = norm[DIN + 2 * s + half];
    }
    stage_weights<FW_THREADS>(S, params);
#pragma unroll
    for (int s = 0; s < DIN / 2; ++s) xn[0][s] = (xn[0][s] - mu[s]) * sd[s];
    __syncthreads();
    if (row0 >= n) return;
    f32x16 h1[2][1];
#pragma unroll
    for (int t = 0; t < 2; ++t) h1[t][0] = load_bias(S.b1[t][half]);
    f32x2 a[2][DIN / 4];
    first_weights<0>(S, a);
    Upper<1> U;
    U.load(S);
    first_layer<0>(a, xn, h1);
    const float v = upper_layers<STORE>(S, params[OFF_B3], h1, U, row0, n, h1t, h2t, [] {});
    if (half == 0 && row < n) y[row] = v;
}

// ---- backward ----
//
// A block of W waves takes chunks of 16 W rows (block b: chunks b, b + G, ...)
// and keeps its partial gradients in accumulators over all of them.  Per chunk:
//   stage   h1, h2 (unit-major), the normalised inputs and dy = 2 (y - t) / n
//           go to LDS; the next chunk's loads are in flight meanwhile;
//   back    d1 = (W2 d2) where h1 > 0, d2 = dy w3 where h2 > 0: a wave owns
//           32 units x 32 rows;
//   grads   dW2 = h1 d2^T, step by step with back: a wave owns one 32 x 32 tile
//           of it, over 64 of the chunk's rows; dW1 = xn d1^T with a row of ones
//           below xn (its product is db1): a wave takes 16 of the rows; db2 and
//           dw3 as a unit's sums per lane.  The waves' sums are added at the end.
// LDS rows are 16 W + 4 floats, so 16-byte reads with one unit per lane hit all
// banks evenly.  Bound by the matrix cores (80 of their 64-cycle steps per wave
// and chunk, 8 us for 60 000 rows) behind the start of the launch and its first
// loads, and the partials' way out.  A training step of 60 000 rows, all its
// kernels: 48.1 us with blocks of four waves, two per CU and twice the partials,
// each weight a round trip of its own and LDS operands read where they were
// used; 40.1 us so.  (With a thread per row and each weight's sum over its rows
// serial in one thread backward alone took 387 us, and one thread per parameter
// adding the 938 partials of 64 rows 220 us.)
// Block partials go to the workspace, part[b * (NP + 1) + p]
// for parameter p and the sum of squared errors at p = NP.
constexpr int BW_XROWS = DIN + 2;         // inputs, ones, zeros
constexpr uint32_t BW_MAX_BLOCKS = 256;  // one per CU

// Waves of a block: eight where four, one to a SIMD, would leave more than one
// chunk to a CU; up to there four spread the rows over more CUs (16 384 rows 26.0
// us a training step, 16 500 30.6 in eight).
inline int bw_waves(uint32_t n) { return n > 64 * BW_MAX_BLOCKS ? 8 : 4; }
inline uint32_t bw_blocks(uint32_t n) {
    const uint32_t rows = 16 * bw_waves(n);
    return (uint32_t)std::min<uint64_t>(((uint64_t)n + rows - 1) / rows, BW_MAX_BLOCKS);
}

template <int W>
struct BackwardLds {
    static constexpr int ROWS = 16 * W, LD = ROWS + 4;
    alignas(16) float w2[2][HID / 8][64][4];  // A operand: W2[32 t + lane%32][2 (4q + e) + lane/32]
    alignas(16) float h1[HID][LD];
    alignas(16) float h2[HID][LD];
    alignas(16) float d1[HID][LD];
    alignas(16) float xs[BW_XROWS][LD];
    alignas(16) float dy[ROWS];
    alignas(16) float w3[3][HID];  // in order; those of unit 2s, 2s + 1 at s
    static_assert(W * (DIN + 1) * HID <= HID * LD, "dW1 partials fit the h1 area");
    static_assert((W - 4) * (16 + 2) * 64 + 2 <= HID * LD, "the upper waves' partials fit the h2 area");
};

// Four consecutive rows of a unit's activations, zero past n.
__device__ __forceinline__ f32x4 load_rows4(const float* __restrict__ p, uint32_t i, uint32_t n) {
    if (i + 4 <= n) return *reinterpret_cast<const f32x4u*>(p + i);
    f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (i + e < n) v[e] = p[i + e];
    return v;
}

template <int W>
__global__ __launch_bounds__(64 * W, 2) void mlp_backward_kernel(
    const float* __restrict__ params, const float* __restrict__ norm, const float* __restrict__ x,
    const float* __restrict__ t, uint32_t n, const float* __restrict__ y, const float* __restrict__ h1t,
    const float* __restrict__ h2t, float* __restrict__ part) {
    constexpr int T = 64 * W, ROWS = 16 * W;
    __shared__ BackwardLds<W> L;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5, l32 = lane & 31;
    const uint32_t chunks = (uint32_t)(((uint64_t)n + ROWS - 1) / ROWS);
    float* w2 = &L.w2[0][0][0][0];
    float wv[HID * HID / T], w3v = 0.0f;
#pragma unroll
    for (int p = 0; p < HID * HID / T; ++p) {
        const int i = tid + T * p;
        const int e = i & 3, ln = (i >> 2) & 63, q = (i >> 8) & 7, tt = i >> 11;
        wv[p] = params[OFF_W2 + (32 * tt + (ln & 31)) * HID + 2 * (4 * q + e) + (ln >> 5)];
    }
    if (tid < HID) w3v = params[OFF_W3 + tid];
    if (tid < L.LD) {
        L.xs[DIN][tid] = 1.0f;
        L.xs[DIN + 1][tid] = 0.0f;
    }

    // Thread's share of a chunk: rows 4 (tid % (4 W)) .. + 3 of units tid / (4 W) + 16 q.
    f32x4 p1[4], p2[4], px;
    float py = 0.0f, pt = 0.0f;
    auto load = [&](uint32_t c) {
        const uint32_t i = c * ROWS + 4 * (tid % (4 * W));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            p1[q] = load_rows4(h1t + (uint64_t)(16 * q + tid / (4 * W)) * n, i, n);
            p2[q] = load_rows4(h2t + (uint64_t)(16 * q + tid / (4 * W)) * n, i, n);
        }
        px = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (tid < ROWS * DIN / 4) {
            const uint32_t r = c * ROWS + tid / (DIN / 4);
            if (r < n) px = *reinterpret_cast<const f32x4u*>(x + (uint64_t)r * DIN + 4 * (tid % (DIN / 4)));
        }
        if (tid < ROWS) {
            const uint32_t r = c * ROWS + tid;
            py = r < n ? y[r] : 0.0f;
            pt = r < n ? t[r] : 0.0f;
        }
    };
    float nmu[4], nsd[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        nmu[e] = norm[4 * (tid % (DIN / 4)) + e];
        nsd[e] = norm[DIN + 4 * (tid % (DIN / 4)) + e];
    }

    const int da = wave & 1, dr = wave >> 1;                       // this wave's tile of d1: units, rows
    const int ta = (wave >> 1) & 1, tj = wave & 1, th = wave >> 2;  // of dW2, over rows 64 th .. + 63
    f32x16 g2, g1[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) g2[r] = g1[0][r] = g1[1][r] = 0.0f;
    float gb2 = 0.0f, gw3 = 0.0f, gb3 = 0.0f, e2 = 0.0f;
    uint32_t c = blockIdx.x;
    load(c);
    __builtin_amdgcn_sched_barrier(0);  // every load is in flight before the first is waited for
#pragma unroll
    for (int p = 0; p < HID * HID / T; ++p) w2[tid + T * p] = wv[p];
    if (tid < HID) {
        L.w3[0][tid] = w3v;
        L.w3[1 + (tid & 1)][tid >> 1] = w3v;
    }
    for (; c < chunks; c += gridDim.x) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            *reinterpret_cast<f32x4*>(&L.h1[16 * q + tid / (4 * W)][4 * (tid % (4 * W))]) = p1[q];
            *reinterpret_cast<f32x4*>(&L.h2[16 * q + tid / (4 * W)][4 * (tid % (4 * W))]) = p2[q];
        }
        if (tid < ROWS * DIN / 4) {
            const int r = tid / (DIN / 4), k = 4 * (tid % (DIN / 4));
            const bool in = c * ROWS + r < n;
#pragma unroll
            for (int e = 0; e < 4; ++e) L.xs[k + e][r] = in ? (px[e] - nmu[e]) * nsd[e] : 0.0f;
        }
        if (tid < ROWS) {
            const float err = py - pt;
            const float dy = 2.0f * err / (float)n;
            L.dy[tid] = dy;
            gb3 += dy;
            e2 += err * err;
        }
        __syncthreads();
        if (c + gridDim.x < chunks) load(c + gridDim.x);

        // d1, units 32 da .. + 31 of rows 32 dr .. + 31, and dW2, which needs no d1;
        // a step's operands are read from LDS during the step before.
        const int row = 32 * dr + l32;
        const float dyr = L.dy[row], w3c = L.w3[0][32 * tj + l32];
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
        struct Step {
            f32x4 w, w3, hr, a, h, dy;
        } st[2];
        auto read = [&](int q, Step& o) {
            o.w = *reinterpret_cast<const f32x4*>(L.w2[da][q][lane]);
            o.w3 = *reinterpret_cast<const f32x4*>(&L.w3[1 + half][4 * q]);
#pragma unroll
            for (int e = 0; e < 4; ++e) o.hr[e] = L.h2[2 * (4 * q + e) + half][row];
            const int k = 64 * th + 8 * q + 4 * half;  // k steps take rows 8q + e and 8q + 4 + e
            o.a = *reinterpret_cast<const f32x4*>(&L.h1[32 * ta + l32][k]);
            o.h = *reinterpret_cast<const f32x4*>(&L.h2[32 * tj + l32][k]);
            o.dy = *reinterpret_cast<const f32x4*>(&L.dy[k]);
        };
        read(0, st[0]);
        float hm[16];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (q < 7) read(q + 1, st[(q + 1) & 1]);
            else
#pragma unroll
                for (int r = 0; r < 16; ++r) hm[r] = L.h1[32 * da + acc_row(r, half)][row];
            __builtin_amdgcn_sched_barrier(0);
            const Step& o = st[q & 1];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc = mfma32(o.w[e], o.hr[e] > 0.0f ? dyr * o.w3[e] : 0.0f, acc);
                const float d2 = o.h[e] > 0.0f ? o.dy[e] * w3c : 0.0f;
                g2 = mfma32(o.a[e], d2, g2);
                gb2 += d2;
                gw3 += o.dy[e] * o.h[e];
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        const int xr = l32 < DIN + 1 ? l32 : DIN + 1, k1 = 16 * wave + 4 * half;
        f32x4 xa[2], dd[2][2];
#pragma unroll
        for (int q = 0; q < 2; ++q) xa[q] = *reinterpret_cast<const f32x4*>(&L.xs[xr][k1 + 8 * q]);
#pragma unroll
        for (int r = 0; r < 16; ++r) L.d1[32 * da + acc_row(r, half)][row] = hm[r] > 0.0f ? acc[r] : 0.0f;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int u = 0; u < 2; ++u) dd[q][u] = *reinterpret_cast<const f32x4*>(&L.d1[32 * u + l32][k1 + 8 * q]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int u = 0; u < 2; ++u) g1[u] = mfma32(xa[q][e], dd[q][u][e], g1[u]);
        __syncthreads();  // the next chunk reuses the LDS
    }

    float* out = part + (uint64_t)blockIdx.x * (NP + 1);
    gb2 += __shfl_xor(gb2, 32);
    gw3 += __shfl_xor(gw3, 32);
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        gb3 += __shfl_xor(gb3, m);
        e2 += __shfl_xor(e2, m);
    }
    float* up = &L.h2[0][0];  // [wave - 4][register, db2, dw3][lane], then the second 64 rows' db3 and error
    float* w1 = &L.h1[0][0];  // [wave][input or ones][unit]
    if (W == 8) {
        if (wave >= 4) {
#pragma unroll
            for (int r = 0; r < 16; ++r) up[((wave - 4) * 18 + r) * 64 + lane] = g2[r];
            up[((wave - 4) * 18 + 16) * 64 + lane] = gb2;
            up[((wave - 4) * 18 + 17) * 64 + lane] = gw3;
        }
        if (wave == 1 && lane == 0) {
            up[4 * 18 * 64] = gb3;
            up[4 * 18 * 64 + 1] = e2;
        }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = acc_row(r, half);
            if (m <= DIN) w1[(wave * (DIN + 1) + m) * HID + 32 * u + l32] = g1[u][r];
        }
    __syncthreads();
    if (wave < 4) {
        if (W == 8) {
#pragma unroll
            for (int r = 0; r < 16; ++r) g2[r] += up[(wave * 18 + r) * 64 + lane];
            gb2 += up[(wave * 18 + 16) * 64 + lane];
            gw3 += up[(wave * 18 + 17) * 64 + lane];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) out[OFF_W2 + (32 * ta + acc_row(r, half)) * HID + 32 * tj + l32] = g2[r];
        if (ta == 0 && half == 0) {
            out[OFF_B2 + 32 * tj + l32] = gb2;
            out[OFF_W3 + 32 * tj + l32] = gw3;
        }
        if (wave == 0 && lane == 0) {
            out[OFF_B3] = W == 8 ? gb3 + up[4 * 18 * 64] : gb3;
            out[NP] = W == 8 ? e2 + up[4 * 18 * 64 + 1] : e2;
        }
    }
    for (int i = tid; i < (DIN + 1) * HID; i += T) {  // W1, then b1 right after it
        float v = 0.0f;
#pragma unroll
        for (int w = 0; w < W; ++w) v += w1[w * (DIN + 1) * HID + i];
        out[i] = v;
    }
}

// Sum of the block partials: 32 parameters per block, so that 158 CUs read; 32
// half-waves each add every 32nd partial (up to eight, their loads all in
// flight), then the half-waves' sums in order.
__global__ __launch_bounds__(1024) void mlp_reduce_kernel(const float* __restrict__ part, uint32_t nblocks,
                                                          uint32_t n, float* __restrict__ grad,
                                                          float* __restrict__ loss) {
    __shared__ float sums[32][32];
    static_assert(BW_MAX_BLOCKS <= 256, "eight partials per half-wave");
    const uint32_t lane = threadIdx.x & 31, g = threadIdx.x >> 5;
    const uint32_t p = blockIdx.x * 32 + lane;
    float v[8];
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q)
        v[q] = p <= NP && g + 32 * q < nblocks ? part[(uint64_t)(g + 32 * q) * (NP + 1) + p] : 0.0f;
    sums[g][lane] = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    __syncthreads();
    if (g == 0 && p <= NP) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < 32; ++w) t += sums[w][lane];
        if (p < NP) grad[p] = t;
        else *loss = t / (float)n;
    }
}

__global__ __launch_bounds__(256) void mlp_adam_kernel(float* __restrict__ p, const float* __restrict__ g,
                                                       float* __restrict__ m, float* __restrict__ v, float lr,
                                                       float b1, float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= NP) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// ---- choose ----
//
// A block owns a contiguous share of the launches and takes them in groups of
// one size, as few as fit the LDS (10 000 launches: 39 in one).  The valid
// (launch, candidate) pairs of a group are packed into one list (in any order: a
// pair's prediction does not depend on its place), the waves evaluate the list
// 64 pairs at a time, the last 32 of an odd share by themselves, under every
// model, and a wave per launch then picks the least mean.  Packing is what keeps
// the matrix cores on real pairs: 96 to 144 of 144 candidates are valid by
// class, and a launch alone would fill its last 64-row tile by a quarter to a
// half.  The first layer's sum over the eight first features is the same for
// all candidates of a launch: it is made once, as the same chain of FMAs, and
// the matrix cores add only the last feature and the schedule (136 of their
// steps per 64 pairs, not 152).  Bound by the matrix cores.
constexpr int CH_THREADS = 512, CH_WAVES = CH_THREADS / 64;
constexpr int CH_CANDS = SPMD_MLP_MAX_CANDS;
constexpr int CH_SHARED = 8;             // features of the shared sum, whole pairs of k steps
constexpr uint32_t CH_MAX_BLOCKS = 256;  // one per CU: two waves per SIMD
constexpr uint32_t CH_GROUP_MAX = 64;
static_assert(SPMD_MLP_NFEAT == CH_SHARED + 1 && DIN == SPMD_MLP_NFEAT + 3 && CH_SHARED % 4 == 0, "first layer's split");
static_assert(CH_CANDS == 256 && CH_GROUP_MAX <= 256, "a list entry is launch * 256 + candidate");

// LDS: the models' weights, then shared sums [model][launch][unit tile][half][16],
// the candidates' normalised inputs (4 floats each), the launches' valid
// candidates (a bit each), means and spreads [launch][c], normalised features
// [launch][9], the list's length and the list.
struct ChooseLayout {
    size_t shared, cand, mask, mean, sd, feat, list, total;
};
__host__ __device__ inline ChooseLayout choose_layout(uint32_t k_models, uint32_t c, uint32_t group) {
    ChooseLayout L;
    L.shared = (size_t)k_models * sizeof(MlpWeights);
    L.cand = L.shared + (size_t)k_models * group * HID * 4;
    L.mask = L.cand + 16 * (size_t)c;
    L.mean = L.mask + 8 * (size_t)group * (CH_CANDS / 64);
    L.sd = L.mean + 4 * (size_t)group * c;
    L.feat = L.sd + 4 * (size_t)group * c;
    L.list = L.feat + 4 * (size_t)group * SPMD_MLP_NFEAT + 4;  // the length sits before the list
    L.total = L.list + 2 * (size_t)group * c;
    return L;
}

struct ChooseArgs {
    uint32_t k_models, c;
    const MlpWeights* W;
    const float *shared, *cand, *feat;
    const uint16_t* list;
    uint32_t group;  // launches the arrays are laid out for
};

// 32 RT pairs from place r0 of the list: the mean over the models of place
// r0 + lane, and its spread.
template <int RT>
__device__ __forceinline__ void choose_rows(const ChooseArgs& A, uint32_t r0, uint32_t rows, float& mean, float& sd) {
    const int lane = (int)lane64(), half = lane >> 5;
    float xn[RT][2];
    uint32_t g[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const uint32_t i = r0 + 32 * rt + (lane & 31);
        const uint32_t id = A.list[i < rows ? i : rows - 1];  // past the end: evaluated, not kept
        g[rt] = id / CH_CANDS;
        const float* s3 = A.cand + 4 * (id % CH_CANDS);
        xn[rt][0] = half ? s3[0] : A.feat[g[rt] * SPMD_MLP_NFEAT + CH_SHARED];
        xn[rt][1] = half ? s3[2] : s3[1];
    }
    // A model's first sums and weights are read while the one before it ends.
    f32x16 h1[2][RT];
    f32x2 a[2][1];
    auto begin = [&](uint32_t mk) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                h1[t][rt] = load_bias(A.shared + (((size_t)mk * A.group + g[rt]) * 4 + 2 * t + half) * 16);
        first_weights<CH_SHARED / 4>(A.W[mk], a);
    };
    // two passes (mean, then squared deviations): the spread of nearly equal
    // predictions keeps its precision
    float pr[SPMD_MLP_MAX_MODELS] = {};
    float s1 = 0.0f;
    begin(0);
#pragma unroll 1
    for (uint32_t mk = 0; mk < A.k_models; ++mk) {
        Upper<RT> U;
        U.load(A.W[mk]);
        __builtin_amdgcn_sched_barrier(0);
        first_layer<CH_SHARED / 4>(a, xn, h1);
        const float y = upper_layers<false>(A.W[mk], A.W[mk].b3, h1, U, 0, 0, nullptr, nullptr, [&] {
            begin(mk + 1 < A.k_models ? mk + 1 : mk);
        });
#pragma unroll
        for (uint32_t i = 0; i < SPMD_MLP_MAX_MODELS; ++i) pr[i] = i == mk ? y : pr[i];
        s1 += y;
    }
    mean = s1 / (float)A.k_models;
    float s2 = 0.0f;
#pragma unroll
    for (uint32_t mk = 0; mk < SPMD_MLP_MAX_MODELS; ++mk) {
        const float d = pr[mk] - mean;
        s2 += mk < A.k_models ? d * d : 0.0f;
    }
    sd = sqrtf(s2 / (float)A.k_models);
}

__global__ __launch_bounds__(CH_THREADS) void mlp_choose_kernel(
    const float* __restrict__ params, uint32_t k_models, const float* __restrict__ norm,
    const float* __restrict__ feats, uint32_t m, const float* __restrict__ cands, uint32_t c,
    const uint8_t* __restrict__ valid, const uint32_t* __restrict__ chunks, float log_slack, uint32_t group,
    uint32_t* __restrict__ best, float* __restrict__ best_pred, float* __restrict__ best_sd) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const ChooseLayout at = choose_layout(k_models, c, group);
    MlpWeights* W = reinterpret_cast<MlpWeights*>(smem);
    float* shared = reinterpret_cast<float*>(smem + at.shared);
    float* cand = reinterpret_cast<float*>(smem + at.cand);
    float* means = reinterpret_cast<float*>(smem + at.mean);
    float* sds = reinterpret_cast<float*>(smem + at.sd);
    float* feat = reinterpret_cast<float*>(smem + at.feat);
    uint64_t* masks = reinterpret_cast<uint64_t*>(smem + at.mask);
    uint16_t* list = reinterpret_cast<uint16_t*>(smem + at.list);
    uint32_t* length = reinterpret_cast<uint32_t*>(smem + at.list - 4);
    const ChooseArgs A{k_models, c, W, shared, cand, feat, list, group};
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (uint32_t k = 0; k < k_models; ++k) stage_weights<CH_THREADS>(W[k], params + k * NP);
    for (uint32_t i = tid; i < 3 * c; i += CH_THREADS) {
        const uint32_t j = i / 3, e = i % 3;
        cand[4 * j + e] = (cands[i] - norm[SPMD_MLP_NFEAT + e]) * norm[DIN + SPMD_MLP_NFEAT + e];
    }
    const uint32_t lo = (uint32_t)((uint64_t)m * blockIdx.x / gridDim.x);
    const uint32_t hi = (uint32_t)((uint64_t)m * (blockIdx.x + 1) / gridDim.x);
    for (uint32_t l0 = lo; l0 < hi; l0 += group) {
        const uint32_t nl = hi - l0 < group ? hi - l0 : group;
        if (tid == 0) *length = 0;
        for (uint32_t i = tid; i < nl * SPMD_MLP_NFEAT; i += CH_THREADS) {
            const uint32_t k = i % SPMD_MLP_NFEAT;
            feat[i] = (feats[(uint64_t)l0 * SPMD_MLP_NFEAT + i] - norm[k]) * norm[DIN + k];
        }
        __syncthreads();
        // a wave per launch: its list entries, a unit per lane of its shared sums
        uint8_t bits[CH_CANDS / 64];
        auto load_valid = [&](uint32_t g) {
#pragma unroll
            for (int q = 0; q < CH_CANDS / 64; ++q) {
                const uint32_t j = 64 * q + lane;
                bits[q] = j < c ? valid[(uint64_t)(l0 + g) * c + j] : 0;
            }
        };
        if (wave < (int)nl) load_valid(wave);
        for (uint32_t mk = 0; mk < k_models; ++mk) {
            const float* w = params + mk * NP + OFF_W1 + lane;
            float wk[CH_SHARED];
#pragma unroll
            for (int k = 0; k < CH_SHARED; ++k) wk[k] = w[k * HID];
            const float b = params[mk * NP + OFF_B1 + lane];
            float* out = shared + (size_t)mk * group * HID + (2 * (lane >> 5) + (lane & 1)) * 16 + ((lane & 31) >> 1);
            for (uint32_t g = wave; g < nl; g += CH_WAVES) {
                float s = b;
#pragma unroll
                for (int k = 0; k < CH_SHARED; ++k) s = __builtin_fmaf(wk[k], feat[g * SPMD_MLP_NFEAT + k], s);
                out[g * HID] = s;
            }
        }
        for (uint32_t g = wave; g < nl; g += CH_WAVES) {
            uint64_t mask[CH_CANDS / 64];
            uint32_t count = 0;
#pragma unroll
            for (int q = 0; q < CH_CANDS / 64; ++q) {
                mask[q] = __builtin_amdgcn_ballot_w64(bits[q] != 0);
                count += (uint32_t)__builtin_popcountll(mask[q]);
            }
            if (g + CH_WAVES < nl) load_valid(g + CH_WAVES);
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(length, count);
            at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
            for (int q = 0; q < CH_CANDS / 64; ++q) {
                const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask[q] >> 32),
                                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)mask[q], 0u));
                if (mask[q] >> lane & 1u) list[at + below] = (uint16_t)(g * CH_CANDS + 64 * q + lane);
                at += (uint32_t)__builtin_popcountll(mask[q]);
                if (lane == 0) masks[g * (CH_CANDS / 64) + q] = mask[q];
            }
        }
        __syncthreads();
        // 32 pairs are a unit of work; a wave's units lie together
        const uint32_t rows = *length, units = (rows + 31) / 32;
        const uint32_t u0 = units * wave / CH_WAVES, u1 = units * (wave + 1) / CH_WAVES;
        auto keep = [&](uint32_t place, float mean, float sd) {
            const uint32_t id = list[place], slot = id / CH_CANDS * c + id % CH_CANDS;
            means[slot] = mean;
            sds[slot] = sd;
        };
        float mean, sd;
        uint32_t u = u0;
        for (; u + 2 <= u1; u += 2) {
            choose_rows<2>(A, 32 * u, rows, mean, sd);
            if (32 * u + lane < rows) keep(32 * u + lane, mean, sd);
        }
        if (u < u1) {
            choose_rows<1>(A, 32 * u, rows, mean, sd);
            if (lane < 32 && 32 * u + lane < rows) keep(32 * u + lane, mean, sd);
        }
        __syncthreads();
        for (uint32_t g = wave; g < nl; g += CH_WAVES) {
            // candidate 64 q + lane in slot q; the tree halves 256 places
            float v[4], sd[4];
            uint32_t id[4], ch[4];
            bool ok[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t j = 64 * q + lane;
                ok[q] = (masks[g * (CH_CANDS / 64) + q] >> lane & 1u) != 0;
                v[q] = ok[q] ? means[g * c + j] : INFINITY;
                sd[q] = ok[q] ? sds[g * c + j] : 0.0f;
                id[q] = ok[q] ? j : 0xFFFFFFFFu;
                ch[q] = 0;
            }
            // a place keeps itself unless the other has fewer chunks, or as
            // many and a smaller mean, or that too and a lower index (in the
            // first pass every chunk count is 0); selects, no branches
            auto take = [](uint32_t& ca, float& a, uint32_t& ia, float& sa, uint32_t cb, float b, uint32_t ib, float sb) {
                const bool other = (cb < ca) | ((cb == ca) & ((b < a) | ((b == a) & (ib < ia))));
                ca = other ? cb : ca;
                a = other ? b : a;
                ia = other ? ib : ia;
                sa = other ? sb : sa;
            };
            auto tree = [&](uint32_t (&tc)[4], float (&tv)[4], uint32_t (&ti)[4], float (&ts)[4]) {
                take(tc[0], tv[0], ti[0], ts[0], tc[2], tv[2], ti[2], ts[2]);
                take(tc[1], tv[1], ti[1], ts[1], tc[3], tv[3], ti[3], ts[3]);
                take(tc[0], tv[0], ti[0], ts[0], tc[1], tv[1], ti[1], ts[1]);
                for (int w = 32; w > 0; w >>= 1)
                    take(tc[0], tv[0], ti[0], ts[0], __shfl_down(tc[0], w), __shfl_down(tv[0], w),
                         __shfl_down(ti[0], w), __shfl_down(ts[0], w));
            };
            float tv[4], ts[4];
            uint32_t ti[4], tc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                tv[q] = v[q];
                ts[q] = sd[q];
                ti[q] = id[q];
                tc[q] = 0;
            }
            tree(tc, tv, ti, ts);
            if (chunks) {
                // Batch-aware second pass: among the candidates whose mean is
                // within log_slack of the least, the fewest chunks wins (then
                // the smaller mean, then the lower index).
                const float thr = __shfl(tv[0], 0) + log_slack;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t j = 64 * q + lane;
                    const bool near = ok[q] && v[q] <= thr;
                    tc[q] = near ? chunks[(uint64_t)(l0 + g) * c + j] : 0xFFFFFFFFu;
                    tv[q] = near ? v[q] : INFINITY;
                    ti[q] = near ? j : 0xFFFFFFFFu;
                    ts[q] = sd[q];
                }
                tree(tc, tv, ti, ts);
            }
            if (lane == 0) {
                best[l0 + g] = ti[0];
                best_pred[l0 + g] = tv[0];
                best_sd[l0 + g] = ts[0];
            }
        }
        __syncthreads();  // the next group reuses the LDS
    }
}

}  // namespace spmd

using namespace spmd;

namespace {
int choose_impl(const float* params, uint32_t k_models, const float* norm, const float* feats, uint32_t m,
                const float* cands, uint32_t c, const uint8_t* valid, const uint32_t* chunks, float log_slack,
                uint32_t* best, float* best_pred, float* best_sd, void* stream);
}  // namespace

extern "C" {

int spmd_mlp_forward(const float* params, const float* norm, const float* x, uint32_t n, float* y, float* h1t,
                     float* h2t, void* stream) {
    if (!params || !norm || (n && (!x || !y)) || (!h1t) != (!h2t)) return SPMD_ERR_ARGS;
    if (!n) return SPMD_OK;
    clear_stale_error();
    constexpr uint32_t per_block = FW_THREADS / 64 * FW_ROWS;
    const dim3 g((uint32_t)(((uint64_t)n + per_block - 1) / per_block)), b(FW_THREADS);
    const hipStream_t s = static_cast<hipStream_t>(stream);
    if (h1t) hipLaunchKernelGGL(mlp_forward_kernel<true>, g, b, 0, s, params, norm, x, n, y, h1t, h2t);
    else hipLaunchKernelGGL(mlp_forward_kernel<false>, g, b, 0, s, params, norm, x, n, y, h1t, h2t);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPMD_OK : hip_fail(e);
}

size_t spmd_mlp_workspace_size(uint32_t n) {
    const size_t nb = (n + MLP_ROWS - 1) / MLP_ROWS;
    return (nb ? nb : 1) * (NP + 1) * sizeof(float);
}

int spmd_mlp_backward(const float* params, const float* norm, const float* x, const float* t, uint32_t n,
                      const float* y, const float* h1t, const float* h2t, float* grad, float* loss, void* workspace,
                      size_t ws_bytes, void* stream) {
    if (!params || !norm || !x || !t || !y || !h1t || !h2t || !grad || !loss || n == 0) return SPMD_ERR_ARGS;
    if (!workspace || ws_bytes < spmd_mlp_workspace_size(n)) return SPMD_ERR_WORKSPACE;
    const uint32_t nb = bw_blocks(n);
    hipStream_t s = static_cast<hipStream_t>(stream);
    float* part = static_cast<float*>(workspace);
    clear_stale_error();
    if (bw_waves(n) == 8)
        hipLaunchKernelGGL(mlp_backward_kernel<8>, dim3(nb), dim3(512), 0, s, params, norm, x, t, n, y, h1t, h2t, part);
    else
        hipLaunchKernelGGL(mlp_backward_kernel<4>, dim3(nb), dim3(256), 0, s, params, norm, x, t, n, y, h1t, h2t, part);
    hipLaunchKernelGGL(mlp_reduce_kernel, dim3((NP + 1 + 31) / 32), dim3(1024), 0, s, part, nb, n, grad, loss);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPMD_OK : hip_fail(e);
}

int spmd_mlp_adam(float* params, const float* grad, float* m, float* v, uint32_t step, float lr, float beta1,
                  float beta2, float eps, void* stream) {
    if (!params || !grad || !m || !v || step == 0) return SPMD_ERR_ARGS;
    const float c1 = 1.0f - powf(beta1, (float)step), c2 = 1.0f - powf(beta2, (float)step);
    clear_stale_error();
    hipLaunchKernelGGL(mlp_adam_kernel, dim3((NP + 255) / 256), dim3(256), 0, static_cast<hipStream_t>(stream),
                       params, grad, m, v, lr, beta1, beta2, eps, c1, c2);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPMD_OK : hip_fail(e);
}

int spmd_mlp_choose_batch(const float* params, uint32_t k_models, const float* norm, const float* feats,
                          uint32_t m, const float* cands, uint32_t c, const uint8_t* valid, const uint32_t* chunks,
                          float slack, uint32_t* best, float* best_pred, float* best_sd, void* stream) {
    if (!chunks || !(slack >= 0.0f) || !(slack < 1e30f)) return SPMD_ERR_ARGS;
    return choose_impl(params, k_models, norm, feats, m, cands, c, valid, chunks, log1pf(slack), best, best_pred,
                       best_sd, stream);
}

int spmd_mlp_choose(const float* params, uint32_t k_models, const float* norm, const float* feats, uint32_t m,
                    const float* cands, uint32_t c, const uint8_t* valid, uint32_t* best, float* best_pred,
                    float* best_sd, void* stream) {
    return choose_impl(params, k_models, norm, feats, m, cands, c, valid, nullptr, 0.0f, best, best_pred, best_sd,
                       stream);
}

}  // extern "C"

namespace {

int choose_impl(const float* params, uint32_t k_models, const float* norm, const float* feats, uint32_t m,
                const float* cands, uint32_t c, const uint8_t* valid, const uint32_t* chunks, float log_slack,
                uint32_t* best, float* best_pred, float* best_sd, void* stream) {
    if (!params || !norm || k_models == 0 || k_models > SPMD_MLP_MAX_MODELS) return SPMD_ERR_ARGS;
    if (c == 0 || c > SPMD_MLP_MAX_CANDS || !cands) return SPMD_ERR_ARGS;
    if (m && (!feats || !valid || !best || !best_pred || !best_sd)) return SPMD_ERR_ARGS;
    if (!m) return SPMD_OK;
    const uint32_t grid = m < CH_MAX_BLOCKS ? m : CH_MAX_BLOCKS;
    // groups of one size, as few as fit the 160 KB LDS (4 models of 256
    // candidates still take 21 launches at a time)
    const uint32_t share = (m + grid - 1) / grid;
    uint32_t fit = CH_GROUP_MAX;
    while (choose_layout(k_models, c, fit).total > 163840) --fit;
    const uint32_t groups = (share + fit - 1) / fit, group = (share + groups - 1) / groups;
    const size_t shm = choose_layout(k_models, c, group).total;
    if (shm > 65536) {  // opted in explicitly
        hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(&mlp_choose_kernel),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
        if (ea != hipSuccess) return hip_fail(ea);
    }
    clear_stale_error();
    hipLaunchKernelGGL(mlp_choose_kernel, dim3(grid), dim3(CH_THREADS), shm, static_cast<hipStream_t>(stream),
                       params, k_models, norm, feats, m, cands, c, valid, chunks, log_slack, group, best, best_pred,
                       best_sd);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? SPMD_OK : hip_fail(e);
}

}  // namespace

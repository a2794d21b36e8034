// cls_gemm.hpp -- block bodies of the GEMM_F32 class: C = A * B, fp32
// row-major, fp32 accumulation on the matrix cores (v_mfma_f32_32x32x2f32: A
// fragment 32 x 2, B fragment 2 x 32, 16 fp32 accumulators per lane).  Two
// forms: K slices staged straight into LDS (whole T x T tiles, enough of them
// to fill the device), and K split over a block's waves (few tiles).
//
// Operand layouts of v_mfma_f32_32x32x2f32 (64 lanes):
//   A: lane l holds A[m = l % 32][k = l / 32]
//   B: lane l holds B[k = l / 32][n = l % 32]
//   D: lane l, register r holds D[m = 8*(r/4) + 4*(l/32) + r%4][n = l % 32]
#pragma once
#include <type_traits>

#include "common.hpp"
#include "warp32.hpp"

namespace spmd {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // any float's address

// ---- Direct-to-LDS form ----
//
// A block of 256 threads (4 waves, 2 x 2) owns a T x T tile of C, each wave a
// (T/2) x (T/2) part of it.  Each K slice (16 deep) goes from HBM to LDS with
// global_load_lds: a lane's V floats land at the instruction's LDS base +
// 4 V * lane, so no register holds the slice and no LDS store is issued, and NS
// slices are in flight at once (a stage each).  V = 4 (16-byte loads) where
// the rows are 16-byte aligned; V = 1 at any other width and alignment, four
// times the loads for the same bytes: 4095^3 at T = 256 1184 us against 1100 for
// 4096^3 with V = 4 (staged through registers element by element it took 1650
// to 1900).  Both operands are laid out for that:
//   A as [m][k] (k contiguous, 64-byte rows); the four 16-byte chunks of
//     row m sit at positions c ^ ((m / 4) % 4), so the 16-lane groups of a
//     16-byte read hit 16 distinct 4-bank groups;
//   B as [k][n]; rows with bit 2 of k set are rotated by 32 columns, so the
//     two half-waves of a read (k and k + 4, same columns) are 32 banks
//     apart.
// The contraction order inside an 8-deep group of k is permuted: in MFMA
// step s, lanes 0-31 take k = 8g + s and lanes 32-63 take k = 8g + 4 + s,
// for A and B alike, so one 16-byte LDS read gives a lane its A values for
// four steps.  A wave waits for its own loads of a slice (vmcnt) and a
// barrier then makes every wave's loads of that slice visible; the stage
// freed by the previous slice is refilled right after that barrier.
// Rows of A past M and columns of B past N are read from the last row or
// column instead (their products land outside C and are not stored); a K
// tail shorter than a slice is loaded through registers with zero fill.
constexpr int GEMM_DMA_KT = 16;

typedef __attribute__((address_space(1))) void gemm_gvoid;
typedef __attribute__((address_space(3))) void gemm_lvoid;

// s_waitcnt: vmcnt <= n, lgkmcnt 0, expcnt not waited (n < 64)
#define GEMM_WAIT_VM(n) __builtin_amdgcn_s_waitcnt(0x70 | ((n) & 15) | (((n) >> 4) << 14))

// The stages are separate LDS arrays passed in by the kernel: the
// compiler then tells a refill from the reads of another stage and does
// not wait for the refill before those reads.
// One load of V floats per lane from `src` to the wave's V * 64 floats at `dst`.
template <int V>
__device__ __forceinline__ void gemm_load_lds(const float* src, float* dst) {
    if constexpr (V == 4) __builtin_amdgcn_global_load_lds((gemm_gvoid*)src, (gemm_lvoid*)dst, 16, 0, 0);
    else __builtin_amdgcn_global_load_lds((gemm_gvoid*)src, (gemm_lvoid*)dst, 4, 0, 0);
}

template <int T, int NS, int V>
__device__ __forceinline__ void gemm_block_dma(const float* __restrict__ A, const float* __restrict__ B,
                                               float* __restrict__ C, uint32_t M, uint32_t N, uint32_t K,
                                               uint32_t bx, uint32_t by, float* S0, float* S1, float* S2,
                                               float* S3) {
    constexpr int KT = GEMM_DMA_KT;
    constexpr int RT = T / 64, WT = T / 2;
    constexpr int CPR = KT / 4;          // 16-byte chunks per A row
    constexpr int RPS = 64 / KT;         // A rows per 64-bank span
    constexpr int NI = T * KT / (256 * V);  // loads per wave per operand per slice
    constexpr int LPW = 2 * NI;          // loads per wave per slice
    constexpr int SA = T * KT;           // floats per operand per stage
    static_assert(V == 1 || V == 4, "floats per load");
    static_assert(NS >= 2 && NS <= 4 && LPW * (NS - 2) < 64, "stage count");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int64_t m0 = (int64_t)by * T, n0 = (int64_t)bx * T;
    const int64_t Mi = M, Ni = N, Ki = K;
    const int nk = (int)(Ki / KT);

    // Per-lane source offsets from the block's slice-0 corner (the launcher
    // checks T * K and KT * N against 2^31).
    const float* Ab = A + m0 * Ki;
    const float* Bb = B + n0;
    int srcA[NI], srcB[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int p = V * (64 * (wave + 4 * i) + lane);  // the lane's first float in the stage
        const int r = p / KT, c = ((p % KT) / 4) ^ ((r / RPS) % CPR);
        const int rr = m0 + r < Mi ? r : (int)(Mi - 1 - m0);  // past M: the last row
        srcA[i] = rr * (int)K + 4 * c + p % 4;
        const int k = p / T;
        const int col = (p % T - ((k & 4) ? 32 : 0) + T) % T;
        const int cc = n0 + col < Ni ? col : (int)(Ni - V - n0);  // past N: the last chunk
        srcB[i] = k * (int)N + cc;
    }
    auto issue = [&](int kt, float* st) {
        const float* a = Ab + (int64_t)kt * KT;
        const float* b = Bb + (int64_t)kt * KT * Ni;
#pragma unroll
        for (int i = 0; i < NI; ++i) gemm_load_lds<V>(a + srcA[i], st + 64 * V * (wave + 4 * i));
#pragma unroll
        for (int i = 0; i < NI; ++i) gemm_load_lds<V>(b + srcB[i], st + SA + 64 * V * (wave + 4 * i));
    };

    f32x16 acc[RT][RT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < RT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    const int kl = lane >> 5, ml = lane & 31;
    const int aswz = (ml / RPS) % CPR;  // rows wm*WT + 32 i + ml share it
    int bcol[RT];
#pragma unroll
    for (int j = 0; j < RT; ++j) bcol[j] = (wn * WT + 32 * j + ml + 32 * kl) % T;
    auto compute = [&](const float* st) {
        const float* as = st;
        const float* bs = st + SA;
#pragma unroll
        for (int g = 0; g < KT / 8; ++g) {
            f32x4 av[RT];
            float bv[RT][4];
#pragma unroll
            for (int i = 0; i < RT; ++i)
                av[i] = *reinterpret_cast<const f32x4*>(as + (wm * WT + 32 * i + ml) * KT + 4 * ((2 * g + kl) ^ aswz));
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int j = 0; j < RT; ++j) bv[j][s] = bs[(8 * g + 4 * kl + s) * T + bcol[j]];
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int i = 0; i < RT; ++i)
#pragma unroll
                    for (int j = 0; j < RT; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i][s], bv[j][s], acc[i][j], 0, 0, 0);
        }
    };
    // Wait until at most `inflight` of this wave's loads are outstanding and
    // its LDS reads are done, then barrier.  The empty asm statements keep
    // the compiler from moving LDS accesses across the barrier; unlike
    // __syncthreads they add no wait for every outstanding load.
    auto barrier_vm = [&](auto inflight) {
        GEMM_WAIT_VM(decltype(inflight)::value);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    auto stage = [&](auto idx) -> float* {
        constexpr int i = decltype(idx)::value;
        if constexpr (i == 0) return S0;
        else if constexpr (i == 1) return S1;
        else if constexpr (i == 2) return S2;
        else return S3;
    };
    // Slice kt is in stage sc: wait for it, refill the stage freed by slice
    // kt - 1 with slice kt + NS - 1, compute.  Inside the main loop every
    // refill is in range, so the wait count holds on every path (a refill
    // that may be skipped would make the compiler wait for all loads).
    auto step = [&](int kt, auto cur, auto full) {
        constexpr int sc = decltype(cur)::value;
        constexpr int sn = (sc + NS - 1) % NS;
        if constexpr (decltype(full)::value) {
            barrier_vm(std::integral_constant<int, LPW * (NS - 2)>());
            issue(kt + NS - 1, stage(std::integral_constant<int, sn>()));
        } else {
            barrier_vm(std::integral_constant<int, 0>());
            if (kt + NS - 1 < nk) issue(kt + NS - 1, stage(std::integral_constant<int, sn>()));
        }
        compute(stage(std::integral_constant<int, sc>()));
    };
    using Full = std::true_type;
    using Tail = std::false_type;
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    // The K tail, shorter than a slice, goes through registers, zero outside the
    // matrices, into stage 0 in the same layouts.  Of 64 x 64 tiles its loads are
    // issued first: they are few, and K is short (4096 x 4096 x 33: 28.7 us, 30.1
    // with them last).
    const int64_t k0 = (int64_t)nk * KT;
    const bool tail = Ki % KT != 0;
    using vec = std::conditional_t<V == 4, f32x4, float>;
    auto tail_a = [&](int p) {
        const int r = p / KT, k = p % KT;
        return m0 + r < Mi && k0 + k < Ki ? *reinterpret_cast<const vec*>(A + (m0 + r) * Ki + k0 + k) : vec{};
    };
    auto tail_b = [&](int p) {
        const int k = p / T, col = p % T;
        return k0 + k < Ki && n0 + col < Ni ? *reinterpret_cast<const vec*>(B + (k0 + k) * Ni + n0 + col) : vec{};
    };
    constexpr bool EARLY = T == 64;
    vec ta[EARLY ? NI : 1], tb[EARLY ? NI : 1];
    if (EARLY && tail) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            ta[i] = tail_a(V * (tid + 256 * i));
            tb[i] = tail_b(V * (tid + 256 * i));
        }
    }
    if (nk > 0) {
        // Slices 0 .. NS - 2, unconditionally (clamped to slice 0), so every
        // path into the loop has the same loads in flight.
        issue(0, S0);
        if constexpr (NS > 2) issue(nk > 1 ? 1 : 0, S1);
        if constexpr (NS > 3) issue(nk > 2 ? 2 : 0, S2);
        int kt = 0;
        for (; kt + 2 * NS - 2 < nk; kt += NS) {
            step(kt, I0(), Full());
            step(kt + 1, I1(), Full());
            if constexpr (NS > 2) step(kt + 2, I2(), Full());
            if constexpr (NS > 3) step(kt + 3, I3(), Full());
        }
        // at most 2 NS - 2 slices remain, the first in stage 0
        if (kt < nk) step(kt, I0(), Tail());
        if (kt + 1 < nk) step(kt + 1, I1(), Tail());
        if constexpr (NS == 3) {
            if (kt + 2 < nk) step(kt + 2, I2(), Tail());
            if (kt + 3 < nk) step(kt + 3, I0(), Tail());
        } else if constexpr (NS == 4) {
            if (kt + 2 < nk) step(kt + 2, I2(), Tail());
            if (kt + 3 < nk) step(kt + 3, I3(), Tail());
            if (kt + 4 < nk) step(kt + 4, I0(), Tail());
            if (kt + 5 < nk) step(kt + 5, I1(), Tail());
        }
        GEMM_WAIT_VM(0);  // the clamped prologue loads too: nothing lands later
        __syncthreads();  // every wave is done reading the stages
    }
    if (tail) {
#pragma unroll(EARLY ? NI : 1)
        for (int i = 0; i < NI; ++i) {
            const int p = V * (tid + 256 * i), r = p / KT, c = p % KT, k = p / T, col = p % T;
            *reinterpret_cast<vec*>(S0 + r * KT + 4 * ((c / 4) ^ ((r / RPS) % CPR)) + c % 4) = EARLY ? ta[EARLY ? i : 0] : tail_a(p);
            *reinterpret_cast<vec*>(S0 + SA + k * T + (col + ((k & 4) ? 32 : 0)) % T) = EARLY ? tb[EARLY ? i : 0] : tail_b(p);
        }
        __syncthreads();
        compute(S0);
    }

#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < RT; ++j) {
            const int64_t col = n0 + wn * WT + j * 32 + ml;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = m0 + wm * WT + i * 32 + (r >> 2) * 8 + kl * 4 + (r & 3);
                if (row < Mi && col < Ni) C[row * Ni + col] = acc[i][j][r];
            }
        }
}


// ---- K-split form (any shape and alignment; few tiles) ----
//
// A block of W waves owns one T x T tile of C, T = 32 RT; every wave computes
// the whole tile over its share of K (8-deep groups dealt round-robin, so the
// waves read neighbouring 32-byte pieces of the same rows of A at the same
// time), and the W partial tiles are added in wave order through LDS at the
// end.  Operands go from global memory straight into registers, D groups
// ahead: no LDS, no barrier and no alignment in the main loop.  Lane l takes
// row l % 32 of A as one 16-byte load of k = 8g + 4 (l / 32) .. + 3 and
// column l % 32 of B as four 4-byte loads (128 bytes contiguous per half-wave);
// k step s multiplies k = 8g + s (lanes 0-31) and 8g + 4 + s.
// Bound by what a CU's vector cache delivers (about 9 bytes a cycle of these
// strided pieces, half to two thirds of what the matrix cores could take), not
// by latency: one, two and four groups ahead and four or eight waves measure
// within 10% of each other.  1000 x 901 x 1111 on 64 x 64 tiles: 25.4 us,
// against 174 us on 128 x 128 tiles staged through registers; 512^3 on 32 x 32
// tiles 5.9 us against 12.1 us on 64 x 64 staged in LDS (64 of 256 CUs busy).
// Rows past M and columns past N are read from the last row or column (their
// products fall outside C and are not stored).
template <int RT, int W>
struct GemmKsplitLds {
    float part[W][16 * RT * RT][64];
};

template <int RT, int W, int D, typename Off>
__device__ __forceinline__ void gemm_block_ksplit(const float* __restrict__ A, const float* __restrict__ B,
                                                  float* __restrict__ C, uint32_t M, uint32_t N, uint32_t K,
                                                  uint32_t bx, uint32_t by, GemmKsplitLds<RT, W>& L) {
    constexpr int T = 32 * RT;
    constexpr int R = 16 * RT * RT;  // accumulators per lane
    static_assert(R % W == 0, "each wave adds R / W of them");
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t m0 = (int64_t)by * T, n0 = (int64_t)bx * T;
    const int64_t Mi = M, Ni = N, Ki = K;
    // Addresses are a wave-uniform base plus the lane's offset from the tile's
    // corner, 32 bits wide where the launcher has checked that they fit.
    const float* Ab = A + m0 * Ki;
    const float* Bb = B + n0;
    Off oa[RT], ob[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i) {
        const int64_t row = m0 + 32 * i + l32 < Mi ? 32 * i + l32 : Mi - 1 - m0;
        const int64_t col = n0 + 32 * i + l32 < Ni ? 32 * i + l32 : Ni - 1 - n0;
        oa[i] = (Off)(4 * (row * Ki + 4 * half));
        ob[i] = (Off)(4 * (col + 4 * half * Ni));
    }
    f32x16 acc[RT][RT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < RT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    f32x4 av[D][RT];
    float bv[D][RT][4];
    auto at = [](const float* base, Off off) {
        return reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + off);
    };
    auto load = [&](const float* pa, const float* pb, f32x4 (&va)[RT], float (&vb)[RT][4]) {
#pragma unroll
        for (int i = 0; i < RT; ++i) va[i] = *reinterpret_cast<const f32x4u*>(at(pa, oa[i]));
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int j = 0; j < RT; ++j) vb[j][s] = *at(pb + s * Ni, ob[j]);
    };
    auto mul = [&](const f32x4 (&va)[RT], const float (&vb)[RT][4]) {
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int j = 0; j < RT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[i][s], vb[j][s], acc[i][j], 0, 0, 0);
    };
    const int64_t full = Ki / 8;                                     // whole groups
    const int64_t mine = full > wave ? (full - wave + W - 1) / W : 0;  // this wave's: wave, wave + W, ...
    if (mine > 0) {
        const float* pa = Ab + 8 * wave;  // the next group to load
        const float* pb = Bb + 8 * wave * Ni;
        int64_t left = mine - 1;  // groups after it: past the wave's last, that one is loaded again
        auto next = [&](f32x4 (&va)[RT], float (&vb)[RT][4]) {
            load(pa, pb, va, vb);
            if (left > 0) {
                pa += 8 * W;
                pb += 8 * W * Ni;
                --left;
            }
        };
#pragma unroll
        for (int d = 0; d < D; ++d) next(av[d], bv[d]);
        int64_t q = 0;
        for (; q + D <= mine; q += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                mul(av[d], bv[d]);
                next(av[d], bv[d]);
                __builtin_amdgcn_sched_barrier(0);  // or the loads of all D groups move behind the products
            }
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (q + d < mine) mul(av[d], bv[d]);
    }
    if (Ki % 8 && full % W == wave) {  // the last K % 8, zero past K
        const int64_t k0 = 8 * full + 4 * half;
        f32x4 va[RT];
        float vb[RT][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const bool in = k0 + s < Ki;
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                va[i][s] = in ? *at(Ab + 8 * full + s, oa[i]) : 0.0f;
                vb[i][s] = in ? *at(Bb + (8 * full + s) * Ni, ob[i]) : 0.0f;
            }
        }
        mul(va, vb);
    }
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < RT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) L.part[wave][(i * RT + j) * 16 + r][lane] = acc[i][j][r];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < R / W; ++e) {
        const int q = wave * (R / W) + e, r = q & 15, ij = q >> 4;
        float v = L.part[0][q][lane];
#pragma unroll
        for (int w = 1; w < W; ++w) v += L.part[w][q][lane];
        const int64_t row = m0 + (ij / RT) * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
        const int64_t col = n0 + (ij % RT) * 32 + l32;
        if (row < Mi && col < Ni) C[row * Ni + col] = v;
    }
}

}  // namespace spmd

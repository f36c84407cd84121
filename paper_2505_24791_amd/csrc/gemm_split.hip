// Float32 projections of whole-sequence passes on the half-precision matrix instruction: C = epi(A W + bias) with both
// operands as sums of two IEEE halves.
//
// A float32 value times a power of two that puts it below 2^15 is hi + lo to 2^-23 of itself (hi the value rounded to a half, lo
// what is left, rounded too); below 2^-16 of the bound the error stays at 2^-40 of it.  A product is then lo hi + hi lo + hi hi, exact in
// the instruction's float32 accumulator; what is left out, lo lo, is below 2^-22 of the product.  The powers of two
// (scale_of) come from the weights alone and bound every value that any input can produce, so nothing overflows.
//
// What bounds it: a tile's walk over k-tiles at small sizes, then the address unit (64 bytes a clock into LDS, half of a 128x64 tile's time) and the power limit of
// the matrix pipe.  A conditioner, us, float32 instruction -> this: 4 layers of width 512, 4096 rows 1208 -> 668; 4 of width 768, 3000 rows 2354 -> 1457; 6 of width
// 256, 8325 rows 1327 -> 986; 2 of width 1024, 1200 rows 917 -> 446.  Its error against 64 bits (2-norm, relative) over these: 0.9e-6 to 1.7e-6 -> 0.6e-6 to 1.1e-6, for
// sixteen products are summed before a result is rounded where the float32 instruction rounds after two.
//
// Layout of a split operand, A [M][K] as well as W transposed [N][K]: a row is K / 16 groups of 64 bytes, a group sixteen consecutive k: sixteen
// hi, then sixteen lo.  A row takes the 4 K bytes of its float32 values, and a group can be converted where it lies.
#include "common.h"
#include <atomic>
#include <cstdint>

namespace sjd {
namespace {

// k-tiles of 32: 128 bytes of a row, a cache line; eight 16-byte chunks: 4 (k / 16) + 2 (lo) + k / 8 % 2
__device__ __forceinline__ int gs_swz(int r) { return ((r >> 1) & 3) | (((r >> 4) & 1) << 2); }

// 64 lanes x 16 bytes from (wave-uniform base) + (32-bit lane offset) to 1 KB of LDS at the wave-uniform byte address
__device__ __forceinline__ void gs_dma(const void *base, uint32_t off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(off), "s"(base) : "memory");
}
template <int N> __device__ __forceinline__ void gs_wait() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory"); }

// A workgroup of four waves (2 x 2) owns a tile of 64 MI rows and 64 NI columns, a wave MI x NI blocks of 32x32; k-tiles in S
// LDS stages filled by LDS-direct loads, requested S - 1 k-tiles ahead.  Every output is a fixed-order sum over k, the same in every tile
// size: a row gives the same bits whatever batch it is computed in.
// LDS: a row of a k-tile is 128 bytes, chunk c in slot c ^ gs_swz(row) (the 16 lanes of one pass of a 16-byte read are rows {0-7, 16-23} or
// {8-15, 24-31}: 8 (row % 2) + slot is distinct over them).
template <int EPI, bool SPLIT_OUT, int MI, int NI, int S>
__global__ __launch_bounds__(256) void gemm_split_kernel(const f16 *__restrict__ A, const f16 *__restrict__ Wt, const float *__restrict__ cs,
                                                         const float *__restrict__ bias, const float *__restrict__ sk, float *C, int M,
                                                         int N, int K, int tiles_n, int n_tiles) {
    constexpr int BM = 64 * MI, BN = 64 * NI;
    constexpr int AQ = 2 * MI, BQ = 2 * NI;                          // loads of 1 KB per wave and k-tile
    constexpr int A_B = BM * 128, STAGE = A_B + BN * 128, LOADS = AQ + BQ;
    extern __shared__ __attribute__((aligned(16))) unsigned char gs_lds[];
    // workgroup ids congruent mod 8 share an XCD: each gets a contiguous run of tiles, column tiles fastest
    const int tile = ((int)blockIdx.x & 7) * ((n_tiles + 7) >> 3) + ((int)blockIdx.x >> 3);
    if (tile >= n_tiles) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    const int tm = tile / tiles_n, m0 = tm * BM, n0 = (tile - tm * tiles_n) * BN;

    uint32_t aoff[AQ], boff[BQ];                             // rows past the end: the last one again, never stored
#pragma unroll
    for (int q = 0; q < AQ; ++q) {
        const int row = 8 * (wave * AQ + q) + (lane >> 3);
        const int rc = m0 + row < M ? row : M - 1 - m0;
        aoff[q] = (uint32_t)rc * (uint32_t)K * 4u + (uint32_t)(((lane & 7) ^ gs_swz(row)) * 16);
    }
#pragma unroll
    for (int q = 0; q < BQ; ++q) {
        const int row = 8 * (wave * BQ + q) + (lane >> 3);
        const int rc = n0 + row < N ? row : N - 1 - n0;
        boff[q] = (uint32_t)rc * (uint32_t)K * 4u + (uint32_t)(((lane & 7) ^ gs_swz(row)) * 16);
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) void *)gs_lds);
    const int KT = K >> 5;
    const char *abase = reinterpret_cast<const char *>(A) + (size_t)m0 * K * 4, *bbase = reinterpret_cast<const char *>(Wt) + (size_t)n0 * K * 4;
    // load q (0 .. LOADS - 1) of a wave for k-tile kt
    auto request1 = [&](int kt, int stage, int q) {
        const int kc = kt < KT ? kt : KT - 1;                        // past the end: into a stage that is not read again
        const uint32_t st = lds0 + (uint32_t)(stage * STAGE);
        if (q < AQ) gs_dma(abase + (size_t)kc * 128, aoff[q < AQ ? q : 0], st + (uint32_t)((wave * AQ + q) * 1024));
        else gs_dma(bbase + (size_t)kc * 128, boff[q < AQ ? 0 : q - AQ], st + (uint32_t)(A_B + (wave * BQ + q - AQ) * 1024));
    };
    auto request = [&](int kt, int stage, int q0, int q1) {
#pragma unroll
        for (int q = 0; q < LOADS; ++q)
            if (q >= q0 && q < q1) request1(kt, stage, q);
    };

    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    struct Frags { f16x8 a[MI][2], b[NI][2]; };                      // [block][hi, lo]
    auto read = [&](Frags &f, int stage, int ks) {
        const unsigned char *As = gs_lds + stage * STAGE + 32 * MI * wm * 128, *Bs = gs_lds + stage * STAGE + A_B + 32 * NI * wn * 128;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int slot = ((4 * ks + 2 * p + g) ^ gs_swz(l32)) << 4;
#pragma unroll
            for (int i = 0; i < MI; ++i) f.a[i][p] = *reinterpret_cast<const f16x8 *>(As + (32 * i + l32) * 128 + slot);
#pragma unroll
            for (int j = 0; j < NI; ++j) f.b[j][p] = *reinterpret_cast<const f16x8 *>(Bs + (32 * j + l32) * 128 + slot);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // The products of a k-step, small ones first, and between them loads q0 .. q1 - 1 of k-tile kt: requested in one go they would hold
    // the wave up until the address unit has taken them all.
    constexpr int HALF = LOADS / 2, NM = 3 * MI * NI;
    auto multiply = [&](const Frags &f, int kt, int stage, int q0) {
        int m = 0;
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    acc[i][j] = Half16<f16>::mfma(f.a[i][p == 0 ? 1 : 0], f.b[j][p == 1 ? 1 : 0], acc[i][j]);
                    const int lo = m * HALF / NM, hi = (m + 1) * HALF / NM;
                    if (hi > lo) {
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int q = 0; q < HALF; ++q)
                            if (q >= lo && q < hi) request1(kt, stage, q0 + q);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    ++m;
                }
        __builtin_amdgcn_sched_barrier(0);
    };
    // this wave's part of the next k-tile has landed (the younger ones may be on their way) and its reads of this one are done; then
    // everyone's, and nobody reads this k-tile's stage any more
    auto next_tile = [&]() {
        gs_wait<(S - 2) * LOADS>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
#pragma unroll
    for (int t = 0; t < S - 1; ++t) request(t, t, 0, LOADS);
    next_tile();
    request(S - 1, S - 1, 0, HALF);
    Frags f0, f1;
    read(f0, 0, 0);
    int stage = 0, prev = S - 1;
    for (int kt = 0; kt < KT; ++kt) {
        read(f1, stage, 1);
        multiply(f0, kt + S - 1, prev, HALF);
        next_tile();
        prev = stage;
        stage = stage + 1 == S ? 0 : stage + 1;
        read(f0, stage, 0);
        multiply(f1, kt + S, prev, 0);
    }
    gs_wait<0>();                            // nothing lands in LDS any more
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    // accumulator register v of block (i, j): row 32 i + 8 (v / 4) + 4 g + v % 4, column 32 j + l32.  A block goes through LDS (a wave's own 32 rows of
    // 36 floats), so that a lane has sixteen consecutive columns of a row: 64 bytes in either output form.
    float *park = reinterpret_cast<float *>(gs_lds) + wave * 32 * 36;
    const int prow = lane >> 1, pc = (lane & 1) * 16;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int gn = n0 + 32 * NI * wn + 32 * j + pc;
        if (n0 + 32 * NI * wn + 32 * j >= N) continue;               // wave-uniform
        const bool whole = gn + 16 <= N && (N & 3) == 0;
        float bv[16], cv[16], sv[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int n = gn + e < N ? gn + e : N - 1;
            bv[e] = bias[n];
            cv[e] = cs[n];
            if (SPLIT_OUT) sv[e] = sk[n];
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) {
#pragma unroll
            for (int v = 0; v < 16; ++v) park[(8 * (v >> 2) + 4 * g + (v & 3)) * 36 + l32] = acc[i][j][v];
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the wave's own rows: no barrier
            __builtin_amdgcn_wave_barrier();
            f32x4 t[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) t[q] = *reinterpret_cast<const f32x4 *>(park + prow * 36 + pc + 4 * q);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_wave_barrier();
            const int gm = m0 + 32 * MI * wm + 32 * i + prow;
            if (gm >= M) continue;
            float *crow = C + (size_t)gm * N + gn;
            if (whole) {
                f32x4 rv[4];
                if (EPI == EPI_BIAS_RESIDUAL)
#pragma unroll
                    for (int q = 0; q < 4; ++q) rv[q] = reinterpret_cast<const f32x4 *>(crow)[q];
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float val = t[q][e] * cv[4 * q + e] + bv[4 * q + e];
                        if (EPI == EPI_BIAS_GELU) val = gelu_erf(val);
                        if (EPI == EPI_BIAS_RESIDUAL) val += rv[q][e];
                        t[q][e] = val;
                    }
                if constexpr (SPLIT_OUT) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        float o[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) o[e] = t[2 * q + (e >> 2)][e & 3] * sv[8 * q + e];
                        store_split8(C, gm, gn + 8 * q, N, o);
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) reinterpret_cast<f32x4 *>(crow)[q] = t[q];
                }
            } else if constexpr (!SPLIT_OUT) {                       // split rows are multiples of 32
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (gn + e < N) {
                        float val = t[e >> 2][e & 3] * cv[e] + bv[e];
                        if (EPI == EPI_BIAS_GELU) val = gelu_erf(val);
                        if (EPI == EPI_BIAS_RESIDUAL) val += crow[e];
                        crow[e] = val;
                    }
            }
        }
    }
}

template <int EPI, bool SPLIT_OUT, int MI, int NI, int S>
void launch_gs(const void *A, const void *Wt, const float *cs, const float *bias, const float *sk, float *C, int M, int N, int K, hipStream_t s) {
    constexpr int BM = 64 * MI, BN = 64 * NI;
    const int tiles_n = (N + BN - 1) / BN, n_tiles = ((M + BM - 1) / BM) * tiles_n;
    constexpr unsigned lds = S * (BM + BN) * 128;
    const auto kern = gemm_split_kernel<EPI, SPLIT_OUT, MI, NI, S>;
    static std::atomic<bool> attr_set{false};   // callers may come from several host threads
    if (lds > 65536 && !attr_set.load(std::memory_order_acquire)) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)((n_tiles + 7) / 8 * 8)), dim3(256), lds, s, (const f16 *)A, (const f16 *)Wt, cs, bias, sk, C, M,
                       N, K, tiles_n, n_tiles);
}

// Tile size: the CUs (256) share the tiles, so a launch takes about ceil(tiles / 256) tiles' worth of work; a smaller tile loads more per
// product.  Two workgroups share a CU, but for 128x128 tiles that are one to a CU at most: four stages then (8192 x 512 x 2048 80.6 -> 55.7 us).
// us as 128x128 / 128x64 / 64x64, M x N x K: 4096 x 1536 x 512 32.8 / 32.6 / 38.1, 4096 x 2048 x 512 39.8 / 42.5 / 56.7, 4096 x 512 x 2048 43.2 / 32.5 / 34.0, 4096 x
// 512 x 512 18.2 / 13.6 / 14.9, 8192 x 1536 x 512 56 / 58 / 71, 8192 x 512 x 2048 56 / 64 / 76, 1024 x 512 x 2048 38 / 25 / 17, 3000 x 3072 x 768 71 / 64 / 82, 3000 x 768 x
// 3072 61.4 / 61.5 / 65.2.
template <int EPI, bool SPLIT_OUT>
void pick_gs(const void *A, const void *Wt, const float *cs, const float *bias, const float *sk, float *C, int M, int N, int K, hipStream_t s) {
    auto cost = [&](int bm, int bn, double weight) {
        const long tiles = (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn);
        return weight * (double)((tiles + 255) / 256) * bm * bn;
    };
    const double c22 = cost(128, 128, 1.0), c21 = cost(128, 64, 1.1), c11 = cost(64, 64, 1.35);
    if (c22 <= c21 && c22 <= c11) {
        if (c22 > 128 * 128) launch_gs<EPI, SPLIT_OUT, 2, 2, 2>(A, Wt, cs, bias, sk, C, M, N, K, s);
        else launch_gs<EPI, SPLIT_OUT, 2, 2, 4>(A, Wt, cs, bias, sk, C, M, N, K, s);
    } else if (c21 <= c11) launch_gs<EPI, SPLIT_OUT, 2, 1, 3>(A, Wt, cs, bias, sk, C, M, N, K, s);
    else launch_gs<EPI, SPLIT_OUT, 1, 1, 5>(A, Wt, cs, bias, sk, C, M, N, K, s);
}

// ---- preparation of the weights -------------------------------------------------------------------
// Bounds that a scale follows: of what a pass stores, so that the product of two scales and a weight by one are float32 numbers, and of a column of weights,
// whose scale only the sums meet.  Outside, zero aside, the flow keeps to the float32 instruction: a scale that stayed behind would cost bits.
constexpr float kLeastBound = 0x1p-40f, kLeastColumn = 0x1p-100f, kLargestBound = 0x1p60f;
// Scale of a channel that is zero for every input (a zero bound), above all others: it may stand beside any other scale, and where scales are
// compared such a channel has no say.
constexpr float kDead = 0x1p56f;

// 2^(15 - e) with 2^(e-1) <= bound < 2^e
__device__ __forceinline__ float scale_of(float bound, float least, int32_t *bad) {
    if (bound == 0.f) return kDead;
    if (!(bound >= least && bound <= kLargestBound)) { *bad = 1; return 1.f; }
    int e;
    (void)frexpf(bound, &e);
    return ldexpf(1.f, 15 - e);
}

// |t| for a bound, t the product of a and b: zero only where one of them is
__device__ __forceinline__ float some(float t, float a, float b) {
    const float least = a != 0.f && b != 0.f ? 0x1p-120f : 0.f;
    return fabsf(t) < least ? least : fabsf(t);          // what is not a number stays so
}

// A workgroup is 64 columns x 16 runs of k; what a column's runs found meets in LDS.
template <class F>
__device__ __forceinline__ float over_k(int K, float (&part)[16][64], bool add, F f) {
    const int cl = threadIdx.x & 63, r = threadIdx.x >> 6;
    float v = 0.f;
#pragma unroll 8
    for (int k = r; k < K; k += 16) { const float t = f(k); v = add ? v + t : fmaxf(v, t); }
    __syncthreads();
    part[r][cl] = v;
    __syncthreads();
    v = part[0][cl];
    for (int q = 1; q < 16; ++q) v = add ? v + part[q][cl] : fmaxf(v, part[q][cl]);
    return v;
}

// sk of LayerNorm's output: |x^ g + be| <= sqrt(K) |g| + |be|
__global__ void ln_scales_kernel(const float *__restrict__ g, const float *__restrict__ be, float *__restrict__ sk, int K, int32_t *bad) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < K) sk[k] = scale_of(1.02f * (sqrtf((float)K) * fabsf(g[k]) + fabsf(be[k])), kLeastBound, bad);
}

// sk of what a projection of LayerNorm's output gives: |sum x^ g w + sum be w + b|, and the squares of x^ add up to K at most
__global__ __launch_bounds__(1024) void ln_projection_scales_kernel(const float *__restrict__ w, int ldw, const float *__restrict__ g,
                                                                    const float *__restrict__ be, const float *__restrict__ b,
                                                                    float *__restrict__ sk, int K, int N, int32_t *bad) {
    __shared__ float part[16][64];
    const int n = blockIdx.x * 64 + (threadIdx.x & 63), nc = n < N ? n : N - 1;
    const float q = over_k(K, part, true, [&](int k) { const float v = w[(size_t)k * ldw + nc], t = g[k] * v; return some(t * t, g[k], v); });
    const float d = over_k(K, part, true, [&](int k) { const float v = w[(size_t)k * ldw + nc]; return some(be[k] * v, be[k], v); });
    if (threadIdx.x < 64 && n < N) sk[n] = scale_of(1.02f * (sqrtf((float)K * q) + d + fabsf(b[n])), kLeastBound, bad);
}

// A head's queries keep their scales; its keys get what makes the product of both the smallest that the 64 pairs of scales have.  A pair with a
// side that is zero adds nothing to a score: it keeps its scales.
__global__ __launch_bounds__(64) void head_scales_kernel(float *sk, float *hs, int W) {
    const int c = blockIdx.x * 64 + threadIdx.x;
    const float q = sk[c], k = sk[W + c];
    const bool live = q != kDead && k != kDead;
    float both = -wave_max(live ? -(q * k) : -INFINITY);
    if (both == INFINITY) both = 1.f;
    if (live) sk[W + c] = both / q;
    if (threadIdx.x == 0) hs[blockIdx.x] = 1.f / both;
}

// Wt[n] = w[., n] / sk times the power of two that brings its largest value below 2^15; cs[n] the inverse of that power
__global__ __launch_bounds__(1024) void split_weights_kernel(const float *__restrict__ w, int ldw, const float *__restrict__ sk,
                                                             f16 *__restrict__ Wt, float *__restrict__ cs, int K, int N, int32_t *bad) {
    __shared__ float part[16][64];
    const int n = blockIdx.x * 64 + (threadIdx.x & 63), nc = n < N ? n : N - 1, r = threadIdx.x >> 6;
    // w / sk; a weight that only ever meets zeros counts as zero (where 0 times it is zero)
    auto value = [&](int k) {
        const float v = w[(size_t)k * ldw + nc], s = sk[k];
        if (s == kDead) return fabsf(v) <= 0x1p120f ? 0.f : v;
        return v * __uint_as_float(0x7F000000u - __float_as_uint(s));        // s is a power of two
    };
    const float top = over_k(K, part, false, [&](int k) { const float t = fabsf(value(k)); return t <= 0x1p120f ? t : 0x1p120f; });
    const float c = scale_of(top, kLeastColumn, bad);
    if (n >= N) return;
    if (r == 0) cs[n] = 1.f / c;
    for (int k = 8 * r; k < K; k += 128) {
        f16x8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float t = keep_f32(value(k + e) * c);
            hi[e] = (f16)t;
            lo[e] = (f16)(t - (float)hi[e]);
        }
        f16x8 *dst = reinterpret_cast<f16x8 *>(Wt + (size_t)n * 2 * K + (k >> 4) * 32 + (k & 8));
        dst[0] = hi;
        dst[2] = lo;
    }
}

// float32 rows to split rows, where they lie
__global__ __launch_bounds__(256) void split_rows_kernel(float *x, const float *__restrict__ sk, size_t n_groups, int groups_per_row) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_groups) return;
    const int c = (int)(i % groups_per_row) * 16;
    f32x4 *p = reinterpret_cast<f32x4 *>(x) + i * 4;
    f32x4 t[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) t[q] = p[q];
#pragma unroll
    for (int q = 0; q < 4; ++q) store_split4(x + i * 16, 0, 4 * q, 16, t[q], *reinterpret_cast<const f32x4 *>(sk + c + 4 * q));
}

}  // namespace

void launch_ln_scales(const float *g, const float *be, float *sk, int K, int32_t *bad, hipStream_t s) {
    hipLaunchKernelGGL(ln_scales_kernel, dim3((K + 255) / 256), dim3(256), 0, s, g, be, sk, K, bad);
}
void launch_ln_projection_scales(const float *w, int ldw, const float *g, const float *be, const float *b, float *sk, int K, int N,
                                 int32_t *bad, hipStream_t s) {
    hipLaunchKernelGGL(ln_projection_scales_kernel, dim3((N + 63) / 64), dim3(1024), 0, s, w, ldw, g, be, b, sk, K, N, bad);
}
void launch_head_scales(float *sk, float *hs, int W, hipStream_t s) {
    hipLaunchKernelGGL(head_scales_kernel, dim3(W / 64), dim3(64), 0, s, sk, hs, W);
}
void launch_split_weights(const float *w, int ldw, const float *sk, void *Wt, float *cs, int K, int N, int32_t *bad, hipStream_t s) {
    hipLaunchKernelGGL(split_weights_kernel, dim3((N + 63) / 64), dim3(1024), 0, s, w, ldw, sk, (f16 *)Wt, cs, K, N, bad);
}
void launch_split_rows(float *x, const float *sk, int rows, int W, hipStream_t s) {
    if (rows <= 0) return;
    const size_t groups = (size_t)rows * (W / 16);
    hipLaunchKernelGGL(split_rows_kernel, dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, s, x, sk, groups, W / 16);
}
void launch_gemm_split(const void *A, const SplitW &w, const float *bias, const float *sk, float *C, int M, int N, int K, Epi epi, hipStream_t s) {
    if (M <= 0 || N <= 0) return;
    switch (epi) {
    case EPI_BIAS:
        if (sk) pick_gs<EPI_BIAS, true>(A, w.wt, w.cs, bias, sk, C, M, N, K, s);
        else pick_gs<EPI_BIAS, false>(A, w.wt, w.cs, bias, nullptr, C, M, N, K, s);
        break;
    case EPI_BIAS_GELU: pick_gs<EPI_BIAS_GELU, true>(A, w.wt, w.cs, bias, sk, C, M, N, K, s); break;
    case EPI_BIAS_RESIDUAL: pick_gs<EPI_BIAS_RESIDUAL, false>(A, w.wt, w.cs, bias, nullptr, C, M, N, K, s); break;
    }
}

}  // namespace sjd

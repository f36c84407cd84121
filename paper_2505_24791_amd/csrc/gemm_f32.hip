// float32 projections (float32 flows, and the refined passes of 16-bit flows): C = epi(A * B + bias).
// Two kernels; the second, on the float32 matrix instruction, takes the shapes it covers.
// The first: 64x64 output tile per workgroup, 4x4 outputs per thread, K walked in index order so that every
// output is one running fused-multiply-add chain over k (no split-K, no atomics): a row's result
// does not depend on the other rows of its tile.
#include "common.h"
#include <cstdint>

namespace sjd {

constexpr int F32_BM = 64, F32_BN = 64, F32_BK = 16;

template <int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float *__restrict__ A, const float *__restrict__ B, int ldb,
                                                       const float *__restrict__ bias, const float *resid, float *C,
                                                       int M, int N, int K) {
    __shared__ float As[F32_BK][F32_BM + 4];
    __shared__ float Bs[F32_BK][F32_BN + 4];
    const int tid = threadIdx.x;
    const int m0 = blockIdx.y * F32_BM, n0 = blockIdx.x * F32_BN;
    const int tx = tid & 15, ty = tid >> 4;  // thread owns rows ty*4.., cols tx*4..
    float acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

    for (int k0 = 0; k0 < K; k0 += F32_BK) {
        // A tile: 64 rows x 16 k = 1024 elements, 4 per thread; stored k-major
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = tid + r * 256;
            const int row = e >> 4, kk = e & 15;
            const int gm = m0 + row, gk = k0 + kk;
            As[kk][row] = (gm < M && gk < K) ? A[(size_t)gm * K + gk] : 0.f;
        }
        // B tile: 16 k x 64 cols
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int e = tid + r * 256;
            const int kk = e >> 6, col = e & 63;
            const int gk = k0 + kk, gn = n0 + col;
            Bs[kk][col] = (gk < K && gn < N) ? B[(size_t)gk * ldb + gn] : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < F32_BK; ++kk) {
            float a[4], b[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx * 4 + j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int gm = m0 + ty * 4 + i;
        if (gm >= M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int gn = n0 + tx * 4 + j;
            if (gn >= N) continue;
            float v = acc[i][j] + bias[gn];
            if (EPI == EPI_BIAS_GELU) v = gelu_erf(v);
            if (EPI == EPI_BIAS_RESIDUAL) v += resid[(size_t)gm * N + gn];
            C[(size_t)gm * N + gn] = v;
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The same product on the float32 matrix instruction (32x32x2), for K % 16 == 0 and rows of B that start on
// 16-byte boundaries.  A workgroup of four waves (2 x 2) owns a tile of 64 MI rows and 64 NI columns, a wave MI x NI
// blocks of 32x32.  k-tiles of 16 in S LDS stages filled by LDS-direct loads, requested S - 1 k-tiles ahead: a k-tile
// is 512 cycles of matrix work per block and a load takes twice that to arrive, so with one k-tile on its way (in
// registers, as before) every k-tile waited.  A lane feeds one value per operand and instruction; step s of lane half
// g stands for k = 8 g + s of the k-tile, so a lane's eight values of A are two 16-byte LDS reads.  Every output is a
// fixed-order sum over k that depends on its own row of A only, the same in every tile size (no split-K): a row gives
// the same bits whatever batch it is computed in.
// LDS: A [rows][16 k], 16-byte chunk c of row r in slot c ^ fm_swz(r) (the 16 lanes of one pass of a 16-byte read are
// rows {0-7, 16-23} or {8-15, 24-31}: 4 (r % 4) + slot is distinct over them); B [16 k][columns], column j of row k at
// j ^ 32 (k / 8), so the two halves of a wave use different banks.
// What bounds it: the float32 matrix pipe (157 TFLOP/s) once the chip is full.
namespace {

__device__ __forceinline__ int fm_swz(int r) { return ((r >> 2) & 1) | (((r >> 4) & 1) << 1); }

// 64 lanes x 16 bytes from (wave-uniform base) + (32-bit lane offset) to 1 KB of LDS at the wave-uniform byte address
__device__ __forceinline__ void fm_dma(const void *base, uint32_t off, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(off), "s"(base) : "memory");
}
template <int N> __device__ __forceinline__ void fm_wait() { asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(N) : "memory"); }

template <int EPI, int MI, int NI, int S>
__global__ __launch_bounds__(256) void gemm_f32_mfma_kernel(const float *__restrict__ A, const float *__restrict__ B, int ldb,
                                                            const float *__restrict__ bias, const float *resid,
                                                            float *C, int M, int N, int K, int tiles_n, int n_tiles) {
    constexpr int BM = 64 * MI, BN = 64 * NI, BK = 16;
    constexpr int A_B = BM * BK * 4, STAGE = A_B + BN * BK * 4, LOADS = MI + NI;   // bytes, bytes, loads per wave and k-tile
    extern __shared__ __attribute__((aligned(16))) unsigned char fm_lds[];
    // workgroup ids congruent mod 8 share an XCD: each gets a contiguous run of tiles, column tiles fastest
    const int tile = ((int)blockIdx.x & 7) * ((n_tiles + 7) >> 3) + ((int)blockIdx.x >> 3);
    if (tile >= n_tiles) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    const int tm = tile / tiles_n, m0 = tm * BM, n0 = (tile - tm * tiles_n) * BN;

    uint32_t aoff[MI], boff[NI];
#pragma unroll
    for (int q = 0; q < MI; ++q) {
        const int row = 16 * (wave * MI + q) + (lane >> 2);
        const int rc = m0 + row < M ? row : M - 1 - m0;              // rows past the end: re-read the last one, never stored
        aoff[q] = ((uint32_t)rc * (uint32_t)K + (uint32_t)(((lane & 3) ^ fm_swz(row)) * 4)) * 4u;
    }
#pragma unroll
    for (int q = 0; q < NI; ++q) {
        const int k = (wave * NI + q) * (4 / NI) + lane / (16 * NI);
        const int gn = n0 + (((lane % (16 * NI)) * 4) ^ ((k >> 3) << 5));
        boff[q] = ((uint32_t)k * (uint32_t)ldb + (uint32_t)(gn < ldb ? gn : 0)) * 4u;   // columns past the end: any, never stored
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)((__attribute__((address_space(3))) void *)fm_lds);
    const int KT = K / BK;
    auto request = [&](int kt, int stage) {
        const int kc = kt < KT ? kt : KT - 1;                        // past the end: into a stage that is not read again
        const float *ab = A + (size_t)m0 * K + (size_t)kc * BK, *bb = B + (size_t)kc * BK * ldb;
        const uint32_t st = lds0 + (uint32_t)(stage * STAGE);
#pragma unroll
        for (int q = 0; q < MI; ++q) fm_dma(ab, aoff[q], st + (uint32_t)((wave * MI + q) * 1024));
#pragma unroll
        for (int q = 0; q < NI; ++q) fm_dma(bb, boff[q], st + (uint32_t)(A_B + (wave * NI + q) * 1024));
    };

    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
#pragma unroll
    for (int t = 0; t < S - 1; ++t) request(t, t);
    int stage = 0;
    for (int kt = 0; kt < KT; ++kt) {
        // this wave's part of k-tile kt has landed (the younger ones may be on their way) and its reads of k-tile kt - 1 are done
        fm_wait<(S - 2) * LOADS>();
        __builtin_amdgcn_s_barrier();        // ... everyone's; and nobody reads the stage of k-tile kt - 1 any more
        asm volatile("" ::: "memory");
        request(kt + S - 1, stage == 0 ? S - 1 : stage - 1);
        const float *As = reinterpret_cast<const float *>(fm_lds + stage * STAGE);
        const float *Bs = reinterpret_cast<const float *>(fm_lds + stage * STAGE + A_B);
        float af[MI][8], bf[NI][8];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int row = 32 * MI * wm + 32 * i + l32;
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                const f32x4 t = *reinterpret_cast<const f32x4 *>(&As[row * BK + (((2 * g + h2) ^ fm_swz(row)) << 2)]);
#pragma unroll
                for (int e = 0; e < 4; ++e) af[i][4 * h2 + e] = t[e];
            }
        }
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int s = 0; s < 8; ++s) bf[j][s] = Bs[(8 * g + s) * BN + ((32 * NI * wn + 32 * j + l32) ^ (g << 5))];
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[i][s], bf[j][s], acc[i][j], 0, 0, 0);
        stage = stage + 1 == S ? 0 : stage + 1;
    }
    fm_wait<0>();                            // nothing lands in LDS after the workgroup has gone
    // accumulator register v of block (i, j): row 32 i + 8 (v / 4) + 4 g + v % 4, column 32 j + l32
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int gn = n0 + 32 * NI * wn + 32 * j + l32;
        if (gn >= N) continue;
        const float bv = bias[gn];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int r0 = m0 + 32 * MI * wm + 32 * i + 4 * g;
            float rv[16];
            if (EPI == EPI_BIAS_RESIDUAL) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int gm = r0 + 8 * (v >> 2) + (v & 3);
                    rv[v] = resid[(size_t)(gm < M ? gm : M - 1) * N + gn];
                }
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int gm = r0 + 8 * (v >> 2) + (v & 3);
                if (gm >= M) continue;
                float val = acc[i][j][v] + bv;
                if (EPI == EPI_BIAS_GELU) val = gelu_erf(val);
                if (EPI == EPI_BIAS_RESIDUAL) val += rv[v];
                C[(size_t)gm * N + gn] = val;
            }
        }
    }
}

template <int EPI, int MI, int NI, int S>
void launch_fm(const float *A, const float *B, int ldb, const float *bias, const float *resid, float *C, int M, int N, int K,
               hipStream_t s) {
    const int tiles_n = (N + 64 * NI - 1) / (64 * NI), n_tiles = ((M + 64 * MI - 1) / (64 * MI)) * tiles_n;
    const unsigned lds = S * (MI + NI) * 4096;
    hipLaunchKernelGGL((gemm_f32_mfma_kernel<EPI, MI, NI, S>), dim3((unsigned)((n_tiles + 7) / 8 * 8)), dim3(256), lds, s, A, B,
                       ldb, bias, resid, C, M, N, K, tiles_n, n_tiles);
}

// Tile size: the CUs (256) share the tiles, and a CU's tiles share its matrix pipes, so a launch takes about
// ceil(tiles / 256) tiles' worth of work; a larger tile reads less LDS per product.  The weights of that (5 and 12 %)
// are what 64x128 and 64x64 lose to 128x128 on launches that fill the chip evenly in all three.
template <int EPI>
void pick_fm(const float *A, const float *B, int ldb, const float *bias, const float *resid, float *C, int M, int N, int K,
             hipStream_t s) {
    auto cost = [&](int bm, int bn, double weight) {
        const long tiles = (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn);
        return weight * (double)((tiles + 255) / 256) * bm * bn;
    };
    const double c22 = cost(128, 128, 1.0), c12 = cost(64, 128, 1.05), c11 = cost(64, 64, 1.12);
    if (c22 <= c12 && c22 <= c11) launch_fm<EPI, 2, 2, 4>(A, B, ldb, bias, resid, C, M, N, K, s);
    else if (c12 <= c11) launch_fm<EPI, 1, 2, 4>(A, B, ldb, bias, resid, C, M, N, K, s);
    else launch_fm<EPI, 1, 1, 5>(A, B, ldb, bias, resid, C, M, N, K, s);
}

}  // namespace

void launch_gemm_f32(const float *A, const float *B, int ldb, const float *bias, const float *resid, float *C, int M, int N,
                     int K, Epi epi, hipStream_t s) {
    if (M <= 0 || N <= 0) return;
    // the choice between the two kernels depends on the matrix shape only, never on the number of rows: a row gives the
    // same bits whatever batch it is computed in
    if (K % 16 == 0 && ldb % 4 == 0 && K >= 16) {
        switch (epi) {
        case EPI_BIAS: pick_fm<EPI_BIAS>(A, B, ldb, bias, resid, C, M, N, K, s); break;
        case EPI_BIAS_GELU: pick_fm<EPI_BIAS_GELU>(A, B, ldb, bias, resid, C, M, N, K, s); break;
        case EPI_BIAS_RESIDUAL: pick_fm<EPI_BIAS_RESIDUAL>(A, B, ldb, bias, resid, C, M, N, K, s); break;
        }
        return;
    }
    dim3 grid((N + F32_BN - 1) / F32_BN, (M + F32_BM - 1) / F32_BM);
    switch (epi) {
        case EPI_BIAS:
            hipLaunchKernelGGL(gemm_f32_kernel<EPI_BIAS>, grid, dim3(256), 0, s, A, B, ldb, bias, resid, C, M, N, K);
            break;
        case EPI_BIAS_GELU:
            hipLaunchKernelGGL(gemm_f32_kernel<EPI_BIAS_GELU>, grid, dim3(256), 0, s, A, B, ldb, bias, resid, C, M, N, K);
            break;
        case EPI_BIAS_RESIDUAL:
            hipLaunchKernelGGL(gemm_f32_kernel<EPI_BIAS_RESIDUAL>, grid, dim3(256), 0, s, A, B, ldb, bias, resid, C, M, N, K);
            break;
    }
}

}  // namespace sjd

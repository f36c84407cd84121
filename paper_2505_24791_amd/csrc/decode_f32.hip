// Single-token steps of the sequential inverse (eq. 5 with the key/value cache of Sec. 3.5) in float32: the float32
// counterparts of the step kernels in decode.hip.  The projections also serve whole-sequence passes of few rows.  A step handles one position of every sample, so a projection
// has as many rows as there are samples, and what it costs is the time until its weights have arrived.
// Rows of activations, LayerNorm parameters and caches start on 16-byte boundaries (blocks of the blob are aligned, widths here are
// multiples of 16); rows of a weight matrix are read by columns and may start anywhere.
#include "common.h"

namespace sjd {

namespace {

// 16x16x4 float32 matrix instruction: lane (r = lane % 16, kg = lane / 16) feeds A[row r][k kg] and B[k kg][col r];
// accumulator register v of that lane is row 4 kg + v, column r.
__device__ __forceinline__ f32x4v mfma4(float a, float b, f32x4v c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

constexpr int S32_NW = 8;     // waves per workgroup; they split k

}  // namespace

// ------------------------------------------------------------------------------------------------
// C[M, N] = epi(LN?(A)[M, K] * Wm[K, N] + bias) for single-token steps; all operands row-major float32.
// A workgroup owns 16 columns and 16*MB rows (blockIdx.y: which rows); its eight waves take an eighth of k each and
// the partial sums meet in LDS, added in wave order.  Inside a wave, instruction e of chunk s stands for
// k = 16 s + 4 kg + e in both operands, so a lane reads its four values of A at once.
// The whole-sequence kernel (gemm_f32.hip), which used to serve these steps, puts all of a narrow product into one
// workgroup that walks k alone: 14 us at k = 128 and 51 us at k = 512 for four rows of the smallest flow
// (width 128), 5 us here; what is left is the launch and two dependent trips to L2.
// LN: the rows of A are normalised on the way in (biased variance, eps 1e-5, mean and centred squares in two passes),
// S = chunks of a wave, K = 128 S.  Without LN, S is 0 and the chunk count is a run-time value (K % 16 == 0).
// A row's sums do not depend on the rows beside it.
template <int MB, int S, int EPI>
__global__ __launch_bounds__(64 * S32_NW) void skinny_f32_kernel(const float *__restrict__ A, const float *__restrict__ g,
                                                                 const float *__restrict__ be, const float *__restrict__ Wm,
                                                                 const float *__restrict__ bias, const float *resid,
                                                                 float *C, int M, int N, int K) {
    constexpr bool LN = S > 0;
    __shared__ f32x4v red[S32_NW * MB * 64];
    __shared__ float stat[S32_NW][MB * 16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = lane & 15, kg = lane >> 4;
    const int n0 = blockIdx.x * 16, row0 = (int)blockIdx.y * 16 * MB;
    const int col = n0 + r, colc = col < N ? col : N - 1;
    const int KC = K >> 4;
    const int s0 = LN ? wave * S : (wave * KC) / S32_NW, s1 = LN ? s0 + S : ((wave + 1) * KC) / S32_NW;
    const float *ap[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        int row = row0 + 16 * i + r;
        row = row < M ? row : M - 1;                 // rows past the end: any row, never stored
        ap[i] = A + (size_t)row * K + 4 * kg;
    }
    const float *bp = Wm + (size_t)(4 * kg) * N + colc;
    const float bv = bias[colc];
    f32x4v acc[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) acc[i] = f32x4v{0.f, 0.f, 0.f, 0.f};
    // the values the finishing waves add: row block i is finished by wave i
    float rv[4] = {0.f, 0.f, 0.f, 0.f};
    if (EPI == EPI_BIAS_RESIDUAL && wave < MB) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = row0 + 16 * wave + 4 * kg + v;
            rv[v] = (row < M && col < N) ? resid[(size_t)row * N + col] : 0.f;
        }
    }

    if constexpr (LN) {
        f32x4 xr[MB][S];
        float w[S][4];
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int i = 0; i < MB; ++i) xr[i][s] = *reinterpret_cast<const f32x4 *>(ap[i] + 16 * (s0 + s));
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) w[s][e] = bp[(size_t)(16 * (s0 + s) + e) * N];
        f32x4 gr[S], br[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            gr[s] = *reinterpret_cast<const f32x4 *>(g + 16 * (s0 + s) + 4 * kg);
            br[s] = *reinterpret_cast<const f32x4 *>(be + 16 * (s0 + s) + 4 * kg);
        }
        float mean[MB], rstd[MB];
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                float t = 0.f;
#pragma unroll
                for (int s = 0; s < S; ++s)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (pass == 0) t += xr[i][s][e];
                        else { const float d = xr[i][s][e] - mean[i]; t = fmaf(d, d, t); }
                    }
                t += __shfl_xor(t, 16, 64);
                t += __shfl_xor(t, 32, 64);
                if (kg == 0) stat[wave][16 * i + r] = t;
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                float t = stat[0][16 * i + r];
#pragma unroll
                for (int q = 1; q < S32_NW; ++q) t += stat[q][16 * i + r];
                if (pass == 0) mean[i] = t / (float)K;
                else rstd[i] = 1.0f / sqrtf(t / (float)K + 1e-5f);
            }
            if (pass == 0) __syncthreads();
        }
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[i] = mfma4((xr[i][s][e] - mean[i]) * rstd[i] * gr[s][e] + br[s][e], w[s][e], acc[i]);
    } else {
        // U chunks in flight: their loads are issued before the first is used
        constexpr int U = 8;
        int s = s0;
        for (; s + U <= s1; s += U) {
            f32x4 a[U][MB];
            float w[U][4];
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int e = 0; e < 4; ++e) w[u][e] = bp[(size_t)(16 * (s + u) + e) * N];
#pragma unroll
                for (int i = 0; i < MB; ++i) a[u][i] = *reinterpret_cast<const f32x4 *>(ap[i] + 16 * (s + u));
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i] = mfma4(a[u][i][e], w[u][e], acc[i]);
        }
        for (; s < s1; s += 2) {
            const int s2 = s + 1 < s1 ? s + 1 : s;
            f32x4 a[2][MB];
            float w[2][4];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int su = u ? s2 : s;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[u][e] = bp[(size_t)(16 * su + e) * N];
#pragma unroll
                for (int i = 0; i < MB; ++i) a[u][i] = *reinterpret_cast<const f32x4 *>(ap[i] + 16 * su);
            }
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (u == 0 || s + 1 < s1)
#pragma unroll
                    for (int i = 0; i < MB; ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[i] = mfma4(a[u][i][e], w[u][e], acc[i]);
        }
    }

#pragma unroll
    for (int i = 0; i < MB; ++i) red[(wave * MB + i) * 64 + lane] = acc[i];
    __syncthreads();
    if (wave < MB && col < N) {
        f32x4v t = red[wave * 64 + lane];
#pragma unroll
        for (int q = 1; q < S32_NW; ++q) t += red[(q * MB + wave) * 64 + lane];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = row0 + 16 * wave + 4 * kg + v;
            if (row >= M) continue;
            float val = t[v] + bv;
            if (EPI == EPI_BIAS_GELU) val = gelu_erf(val);
            if (EPI == EPI_BIAS_RESIDUAL) val += rv[v];
            C[(size_t)row * N + col] = val;
        }
    }
}

template <int MB, int S>
static void launch_skinny_f32_one(const float *A, const float *g, const float *be, const float *Wm, const float *bias,
                                  const float *resid, float *C, int M, int N, int K, Epi epi, hipStream_t s) {
    const dim3 grid((N + 15) / 16, (M + 16 * MB - 1) / (16 * MB)), block(64 * S32_NW);
    switch (epi) {
    case EPI_BIAS: hipLaunchKernelGGL((skinny_f32_kernel<MB, S, EPI_BIAS>), grid, block, 0, s, A, g, be, Wm, bias, resid, C, M, N, K); break;
    case EPI_BIAS_GELU: hipLaunchKernelGGL((skinny_f32_kernel<MB, S, EPI_BIAS_GELU>), grid, block, 0, s, A, g, be, Wm, bias, resid, C, M, N, K); break;
    case EPI_BIAS_RESIDUAL: hipLaunchKernelGGL((skinny_f32_kernel<MB, S, EPI_BIAS_RESIDUAL>), grid, block, 0, s, A, g, be, Wm, bias, resid, C, M, N, K); break;
    }
}

bool skinny_f32_ln_ok(int K) { return K == 128 || K == 256 || K == 512 || K == 768 || K == 1024; }

void launch_skinny_f32(const float *A, const float *g, const float *be, const float *Wm, const float *bias,
                       const float *resid, float *C, int M, int N, int K, Epi epi, hipStream_t s) {
    if (M <= 0 || N <= 0) return;
    // one row block for up to 16 rows, two (sharing the weight values of a column) above
#define SJD_S32(Sv) do { if (M <= 16) launch_skinny_f32_one<1, Sv>(A, g, be, Wm, bias, resid, C, M, N, K, epi, s); \
                         else launch_skinny_f32_one<2, Sv>(A, g, be, Wm, bias, resid, C, M, N, K, epi, s); } while (0)
    if (!g) { SJD_S32(0); return; }
    switch (K) {
    case 128: SJD_S32(1); break;
    case 256: SJD_S32(2); break;
    case 512: SJD_S32(4); break;
    case 768: SJD_S32(6); break;
    case 1024: SJD_S32(8); break;
    default: break;              // skinny_f32_ln_ok() keeps other widths away
    }
#undef SJD_S32
}

// ------------------------------------------------------------------------------------------------
// Single-token attention against the float32 cache.  One workgroup of 256 threads per (sample, head); LPK = dh / 4
// lanes share a key, four values each, so 256 / LPK keys are walked at a time, each lane of a key reading 16
// consecutive bytes (the row-wise kernel of attention.hip gives a whole key to a lane: 64 rows apart between
// neighbouring lanes, and one dependent load after the other).  Position t = *t_dev: this step's k, v are
// appended to the cache and used from the fresh row.  Scores in LDS; four keys in flight per thread.
template <int LPK>
__global__ __launch_bounds__(256) void decode_attention_f32_kernel(const float *__restrict__ qkv, float *kcache, float *vcache,
                                                                   float *__restrict__ o, const int32_t *__restrict__ t_dev,
                                                                   int T, int H, float scale) {
    constexpr int DH = 4 * LPK, G = 256 / LPK, U = 4;
    extern __shared__ float sc[];                 // [T] scores
    __shared__ float wmax[4], wsum[4];
    __shared__ float opart[4][DH];
    const int t = *t_dev;
    const int W = H * DH;
    const int h = blockIdx.x % H, b = blockIdx.x / H;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int dc = tid % LPK, sg = tid / LPK;
    const float *row = qkv + (size_t)b * 3 * W + h * DH + dc * 4;
    const f32x4 q4 = *reinterpret_cast<const f32x4 *>(row);
    const float *kf = row + W, *vf = row + 2 * W;                        // this thread's part of the fresh k, v
    float *kc = kcache + (size_t)b * T * W + h * DH + dc * 4, *vc = vcache + (size_t)b * T * W + h * DH + dc * 4;
    if (sg == 0) {
        *reinterpret_cast<f32x4 *>(kc + (size_t)t * W) = *reinterpret_cast<const f32x4 *>(kf);
        *reinterpret_cast<f32x4 *>(vc + (size_t)t * W) = *reinterpret_cast<const f32x4 *>(vf);
    }
    const int n = t + 1;
    float mx = -INFINITY;
    for (int s0 = sg; s0 < n; s0 += G * U) {
        f32x4 k4[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + G * u;
            k4[u] = *reinterpret_cast<const f32x4 *>(s < t ? kc + (size_t)s * W : kf);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + G * u;
            if (s < n) {                           // the lanes of a key agree on s
                float d = fmaf(q4[3], k4[u][3], fmaf(q4[2], k4[u][2], fmaf(q4[1], k4[u][1], q4[0] * k4[u][0])));
#pragma unroll
                for (int off = 1; off < LPK; off <<= 1) d += __shfl_xor(d, off, 64);
                d *= scale;
                if (dc == 0) sc[s] = d;
                mx = fmaxf(mx, d);
            }
        }
    }
    mx = wave_max(mx);
    if (lane == 0) wmax[wave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float psum = 0.f;
    for (int s0 = sg; s0 < n; s0 += G * U) {
        f32x4 v4[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + G * u;
            v4[u] = *reinterpret_cast<const f32x4 *>(s < t ? vc + (size_t)s * W : vf);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = s0 + G * u;
            if (s < n) {
                const float p = expf(sc[s] - mx);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] = fmaf(p, v4[u][e], acc[e]);
                psum += p;
            }
        }
    }
    // the key groups of a wave, then the four waves in order
#pragma unroll
    for (int off = LPK; off < 64; off <<= 1) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], off, 64);
        psum += __shfl_xor(psum, off, 64);
    }
    if (lane < LPK) {
#pragma unroll
        for (int e = 0; e < 4; ++e) opart[wave][lane * 4 + e] = acc[e];
        if (lane == 0) wsum[wave] = psum;
    }
    __syncthreads();
    if (tid < DH) {
        const float den = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
        o[(size_t)b * W + h * DH + tid] = (((opart[0][tid] + opart[1][tid]) + opart[2][tid]) + opart[3][tid]) / den;
    }
}

bool decode_attention_f32_ok(int dh) { return dh == 16 || dh == 32 || dh == 64 || dh == 128; }

void launch_decode_attention_f32(const float *qkv, float *kcache, float *vcache, float *o, const int32_t *t_dev, int B, int T,
                                 int H, int dh, hipStream_t s) {
    if (B <= 0) return;
    const float scale = 1.0f / sqrtf((float)dh);
    const dim3 grid(B * H), block(256);
    const size_t lds = (size_t)T * sizeof(float);
    switch (dh) {
    case 16: hipLaunchKernelGGL(decode_attention_f32_kernel<4>, grid, block, lds, s, qkv, kcache, vcache, o, t_dev, T, H, scale); break;
    case 32: hipLaunchKernelGGL(decode_attention_f32_kernel<8>, grid, block, lds, s, qkv, kcache, vcache, o, t_dev, T, H, scale); break;
    case 64: hipLaunchKernelGGL(decode_attention_f32_kernel<16>, grid, block, lds, s, qkv, kcache, vcache, o, t_dev, T, H, scale); break;
    case 128: hipLaunchKernelGGL(decode_attention_f32_kernel<32>, grid, block, lds, s, qkv, kcache, vcache, o, t_dev, T, H, scale); break;
    default: break;              // decode_attention_f32_ok() keeps other head sizes away
    }
}

}  // namespace sjd

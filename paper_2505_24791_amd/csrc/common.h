// Shared declarations of the HIP library: element types, launchers of every kernel family.
// gfx950 only (64-wide wavefronts, MFMA, 160 KB LDS per CU).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sjd {

typedef __bf16 bf16;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16;
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kWave = 64;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

template <typename T> __device__ __forceinline__ float to_f32(T v);
template <> __device__ __forceinline__ float to_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ float to_f32<bf16>(bf16 v) { return (float)v; }
template <> __device__ __forceinline__ float to_f32<f16>(f16 v) { return (float)v; }
template <typename T> __device__ __forceinline__ T from_f32(float v);
template <> __device__ __forceinline__ f16 from_f32<f16>(float v) { return (f16)v; }
template <> __device__ __forceinline__ float from_f32<float>(float v) { return v; }
template <> __device__ __forceinline__ bf16 from_f32<bf16>(float v) { return (bf16)v; }

// The two 16-bit operand types of the MFMA kernels: vectors of 4 / 8 elements and the
// 32x32x16 matrix instruction with float32 accumulation.
template <typename HT> struct Half16;
template <> struct Half16<bf16> {
    typedef bf16x4 v4;
    typedef bf16x8 v8;
    static __device__ __forceinline__ f32x16 mfma(v8 a, v8 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    }
    // c + the sum of the eight values of p, in float32 (two values per instruction)
    static __device__ __forceinline__ float add_all(v8 p, float c) {
        typedef __bf16 v2 __attribute__((ext_vector_type(2)));
        const v2 one = {(__bf16)1.f, (__bf16)1.f};
        c = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p, p, 0, 1), one, c, false);
        c = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p, p, 2, 3), one, c, false);
        c = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p, p, 4, 5), one, c, false);
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(p, p, 6, 7), one, c, false);
    }
    // the dot product of eight pairs, exact products summed in float32
    static __device__ __forceinline__ float dot(v8 a, v8 b) {
        float c = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 0, 1), __builtin_shufflevector(b, b, 0, 1), 0.f, false);
        c = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 2, 3), __builtin_shufflevector(b, b, 2, 3), c, false);
        c = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 4, 5), __builtin_shufflevector(b, b, 4, 5), c, false);
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(a, a, 6, 7), __builtin_shufflevector(b, b, 6, 7), c, false);
    }
};
template <> struct Half16<f16> {
    typedef f16x4 v4;
    typedef f16x8 v8;
    static __device__ __forceinline__ f32x16 mfma(v8 a, v8 b, f32x16 c) {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ float add_all(v8 p, float c) {
        typedef _Float16 v2 __attribute__((ext_vector_type(2)));
        const v2 one = {(_Float16)1.f, (_Float16)1.f};
        c = __builtin_amdgcn_fdot2(__builtin_shufflevector(p, p, 0, 1), one, c, false);
        c = __builtin_amdgcn_fdot2(__builtin_shufflevector(p, p, 2, 3), one, c, false);
        c = __builtin_amdgcn_fdot2(__builtin_shufflevector(p, p, 4, 5), one, c, false);
        return __builtin_amdgcn_fdot2(__builtin_shufflevector(p, p, 6, 7), one, c, false);
    }
    // the dot product of eight pairs, exact products summed in float32
    static __device__ __forceinline__ float dot(v8 a, v8 b) {
        float c = __builtin_amdgcn_fdot2(__builtin_shufflevector(a, a, 0, 1), __builtin_shufflevector(b, b, 0, 1), 0.f, false);
        c = __builtin_amdgcn_fdot2(__builtin_shufflevector(a, a, 2, 3), __builtin_shufflevector(b, b, 2, 3), c, false);
        c = __builtin_amdgcn_fdot2(__builtin_shufflevector(a, a, 4, 5), __builtin_shufflevector(b, b, 4, 5), c, false);
        return __builtin_amdgcn_fdot2(__builtin_shufflevector(a, a, 6, 7), __builtin_shufflevector(b, b, 6, 7), c, false);
    }
};

typedef float f32x4v __attribute__((ext_vector_type(4)));

template <typename HT> struct Mfma16;
template <> struct Mfma16<bf16> {
    static __device__ __forceinline__ f32x4v run(bf16x8 a, bf16x8 b, f32x4v c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct Mfma16<f16> {
    static __device__ __forceinline__ f32x4v run(f16x8 a, f16x8 b, f32x4v c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
};

// Fragment-major layout of a [rows, K] operand of the 16x16x32 MFMA: the 64 x 8 elements one wave
// feeds to one instruction (lane = 16*(k%32/8) + row%16 holds 8 consecutive k) are contiguous,
// fragment (row/16, k/32) after fragment.  KS = K/32.  Returns the element index of (row, k).
__device__ __forceinline__ size_t frag_off(int row, int k, int KS) {
    return ((((size_t)(row >> 4) * KS + (k >> 5)) * 64 + (((k & 31) >> 3) << 4) + (row & 15)) << 3) + (k & 7);
}

__device__ __forceinline__ float gelu_erf(float v) { return 0.5f * v * (1.0f + erff(v * 0.70710678118654752440f)); }

// A float32 value that is about to be rounded to 16 bits, made opaque to the compiler.  Otherwise it
// folds the fma that produces the value into the conversion (v_fma_mix: one rounding instead of
// two) for some elements of an unrolled loop and not for others, and two kernels that compute the
// same thing differ in the last bit of a few results per hundred thousand.
__device__ __forceinline__ float keep_f32(float v) {
    asm("" : "+v"(v));
    return v;
}

// GELU (erf form) for results that are stored in 16 bits: gelu(v) = max(v, 0) - |v| Phi(-|v|), Phi the normal
// distribution function, and log2 Phi(-t) is smooth enough for one polynomial, degree 8, fitted on 0 <= t <= 6 with the error
// of Phi weighted by max(t, 1).  Evaluated in float32 that weighted error is at most 5.3e-8: an absolute bound, for in the
// negative tail the relative error grows (0.6 % of a result of 1e-5, 8 % of one of 1e-8).  Beyond 6 the negative leading
// coefficient carries Phi to zero.  The rational-times-exponential formula of Abramowitz & Stegun 7.1.26 has 7.5e-8 in Phi (and
// a larger error in every range of v), takes nineteen issue slots where this takes fifteen, and a reciprocal as well; the slots
// are what the epilogue of the MLP input projection costs (M = 32768, N = 4096, K = 1024: 289 us with that formula, 277 now).
// The IEEE minimum with 16 (Phi is zero long before; a NaN stays a NaN) keeps |v| Phi(-|v|) of +inf from being inf * 0, for 5 of
// those 277 us; -inf gives NaN, as 0.5 v (1 + erf(v / sqrt 2)) does.
__device__ __forceinline__ float gelu_erf_h16(float v) {
    const float t = fabsf(__builtin_elementwise_minimum(v, 16.f));
    float p = fmaf(-2.27592182e-06f, t, 3.29686736e-05f);
    p = fmaf(p, t, -0.000157282251f);
    p = fmaf(p, t, -0.000202469484f);
    p = fmaf(p, t, 0.00714276778f);
    p = fmaf(p, t, -0.0525464229f);
    p = fmaf(p, t, -0.459193051f);
    p = fmaf(p, t, -1.15110695f);
    p = fmaf(p, t, -0.99999994f);
    return keep_f32(fmaf(-t, __builtin_amdgcn_exp2f(p), fmaxf(v, 0.f)));
}

// Split rows (gemm_split.hip): a row of W values, W % 16 == 0, takes the 4 W bytes of its float32 values; sixteen consecutive
// values are 64 bytes, sixteen halves hi, then sixteen lo, value * s = hi + lo with a power of two s.
__device__ __forceinline__ void store_split4(void *base, size_t row, int col, int W, f32x4 v, f32x4 s) {
    f16x4 hi, lo;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const float t = keep_f32(v[e] * s[e]);   // or hi may be rounded from the unrounded product, and lo be taken from another hi
        hi[e] = (f16)t;
        lo[e] = (f16)(t - (float)hi[e]);
    }
    char *p = (char *)base + (row * W + (col & ~15)) * 4 + (col & 15) * 2;
    *reinterpret_cast<f16x4 *>(p) = hi;
    *reinterpret_cast<f16x4 *>(p + 32) = lo;
}

// eight columns, in 16-byte stores
__device__ __forceinline__ void store_split8(void *base, size_t row, int col, int W, const float (&v)[8]) {   // values with their scales
    f16x8 hi, lo;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float t = keep_f32(v[e]);
        hi[e] = (f16)t;
        lo[e] = (f16)(t - (float)hi[e]);
    }
    char *p = (char *)base + (row * W + (col & ~15)) * 4 + (col & 15) * 2;
    *reinterpret_cast<f16x8 *>(p) = hi;
    *reinterpret_cast<f16x8 *>(p + 32) = lo;
}

// Row -> (sample, token) mapping shared by the embedding and the epilogues.  A whole-sequence pass
// runs on `rows_per_sample = T` rows per active sample; a single-token step on one row per sample.
struct RowMap {
    const int32_t *active;  // [n_rows / rows_per_sample] sample indices, or nullptr for the identity
    int32_t rows_per_sample;
    int32_t t0;             // processing-order position of a sample's first row
    int32_t T;              // tokens per sample
    int32_t reversed;       // 1: processing position p is canonical token T-1-p
};

// Epilogue selector of the dense projections.
enum Epi : int {
    EPI_BIAS = 0,          // out = acc + bias
    EPI_BIAS_GELU = 1,     // out = gelu(acc + bias)
    EPI_BIAS_RESIDUAL = 2, // out(float) = resid(float) + acc + bias, in place allowed
};

// ---- launchers (all asynchronous on `s`) ---------------------------------------------------

// h[m, :] = x[b, tok, :] * w_in + b_in + pos[p, :]
void launch_embed(const float *x, const float *w_in, const float *b_in, const float *pos, float *h, int n_rows,
                  int D, int W, RowMap map, hipStream_t s);

// y = LayerNorm(x) * g + b over rows of width W (biased variance, eps 1e-5); OutT float, bf16 or f16
template <typename OutT>
void launch_layernorm(const float *x, const float *g, const float *b, OutT *y, int n_rows, int W, hipStream_t s);

// float32 projection: C[M,N] = epi(A[M,K] * B[K,N] + bias), rows of B ldb floats apart; A and B 16-byte aligned
void launch_gemm_f32(const float *A, const float *B, int ldb, const float *bias, const float *resid, float *C, int M, int N,
                     int K, Epi epi, hipStream_t s);

// The same on split operands (gemm_split.hip), K % 32 == 0: A [M, K] split rows with the scales its producer was given (one
// power of two per k), the weights as launch_split_weights leaves them.  EPI_BIAS_RESIDUAL (C is the residual, in place) and EPI_BIAS
// without sk give float32; EPI_BIAS_GELU and EPI_BIAS with sk give split rows with the scales sk [N], N % 32 == 0.
struct SplitW { const void *wt; const float *cs; };   // [N][K] split rows; [N] what takes the scales out of a sum again
void launch_gemm_split(const void *A, const SplitW &w, const float *bias, const float *sk, float *C, int M, int N, int K, Epi epi,
                       hipStream_t s);
void launch_layernorm_split(const float *x, const float *g, const float *b, const float *sk, void *y, int n_rows, int W, hipStream_t s);
void launch_split_rows(float *x, const float *sk, int rows, int W, hipStream_t s);   // float32 rows to split rows in place
// Scales of LayerNorm's output, and of a projection of it ([K, N], rows ldw floats apart); weights with the scales sk of their k.  *bad is set where a
// bound is out of range: the float32 instruction then.
void launch_ln_scales(const float *g, const float *be, float *sk, int K, int32_t *bad, hipStream_t s);
void launch_ln_projection_scales(const float *w, int ldw, const float *g, const float *be, const float *b, float *sk, int K, int N,
                                 int32_t *bad, hipStream_t s);
// Heads of 64: the keys' scales (sk [3 W]) such that query times key has one scale 1 / hs[h] for all d of a head
void launch_head_scales(float *sk, float *hs, int W, hipStream_t s);
void launch_split_weights(const float *w, int ldw, const float *sk, void *Wt, float *cs, int K, int N, int32_t *bad, hipStream_t s);

// 16-bit MFMA projection (HT = bf16 or f16): C[M,N] = epi(A[M,K] * Bt[N,K]^T + bias); Bt holds the
// weight transposed, K contiguous, with at least round_up(N, 256) rows (zero filled).  K % 64 == 0.
// OutT = HT (EPI_BIAS, EPI_BIAS_GELU) or float (EPI_BIAS, EPI_BIAS_RESIDUAL).
// kernel: 0 = chosen by shape; 1 = 256x128x32 staged through registers; 2 = 256x256x64 LDS-direct;
// 3 = 128x128x64; 4 = the persistent eight-wave kernel of gemm_p8.hip where it applies (else as 0)
// (the explicit choices exist so that each kernel can be checked on small shapes).
template <typename HT, typename OutT>
void launch_gemm_h16(const HT *A, const HT *Bt, const float *bias, const float *resid, OutT *C, int M, int N, int K,
                     Epi epi, hipStream_t s, int kernel = 0);

// Persistent eight-wave projection (gemm_p8.hip): the same contract as launch_gemm_h16 (resid, when given, is C
// itself: the float32 stream is updated in place) for K % 64 == 0, K >= 128 and N % 256 == 0; bit-identical to the tile kernels.
bool gemm_p8_applicable(int M, int N, int K);
template <typename HT, typename OutT>
void launch_gemm_p8(const HT *A, const HT *Bt, const float *bias, OutT *C, int M, int N, int K, Epi epi, hipStream_t s);

// MLP-input projection with GELU for launches that fill the chip (gemm_duo.hip): C[M,N] (16-bit) = gelu(A[M,K] * W + bias), W in the
// fragment order of the 32x32x16 instruction (launch_weights_to_frag32 from the transposed [N, K] copy); bit-identical to launch_gemm_h16.
// For launches that gemm_duo_applicable() (gemm_rules.h) admits.
template <typename HT>
void launch_gemm_duo_gelu(const HT *A, const HT *Wf, const float *bias, HT *C, int M, int N, int K, hipStream_t s);

// Activation-stationary projections for K = 512 (gemm_panel.hip).  Wf: the weight in the fragment order of
// the 32x32x16 instruction (launch_weights_to_panel_frag from the transposed [N, 512] copy; N % 256 == 0).
//   launch_ln_gemm_panel:    C[M,N] (16-bit) = epi(LayerNorm(H[M,512]; g, b) * W + bias), epi = EPI_BIAS or EPI_BIAS_GELU
//   launch_gemm_panel_resid: H[M,N] (float32) += A[M,512] * W + bias
// Bit-identical to launch_layernorm + launch_gemm_h16.  gemm_panel_applicable: the shape is covered
// (out_bytes: element size of the output).
bool gemm_panel_applicable(int M, int N, int K, int out_bytes);
template <typename HT> void launch_weights_to_panel_frag(const HT *wt, HT *dst, int N, hipStream_t s);
template <typename HT>
void launch_ln_gemm_panel(const float *H, const float *g, const float *b, const HT *Wf, const float *bias, HT *C, int M,
                          int N, Epi epi, hipStream_t s);
template <typename HT>
void launch_gemm_panel_resid(const HT *A, const HT *Wf, const float *bias, float *H, int M, int N, hipStream_t s);

// Residual projection for long k (gemm_stream.hip): H[M,N] (float32) += A[M,K] * W + bias with the left operand
// streamed through LDS in chunks of 256 k and the weights in the fragment order of the 32x32x16 instruction
// (launch_weights_to_frag32 from the transposed [N, K] copy).  K % 512 == 0, N % 256 == 0; bit-identical to
// launch_gemm_h16.
bool gemm_stream_applicable(int M, int N, int K);
template <typename HT> void launch_weights_to_frag32(const HT *wt, HT *dst, int N, int K, hipStream_t s);
template <typename HT>
void launch_gemm_stream_resid(const HT *A, const HT *Wf, const float *bias, float *H, int M, int N, int K, hipStream_t s);

// Causal attention, one wave per (sample, head, query row); works for any shape and both types.
// q rows: q + (sample*q_rows_per_sample + r) * q_stride; row r (processing position t0 + r) attends
// keys 0..t0+r-mask_o found at k + sample_index*kv_sample_stride + key*kv_stride (+ head*dh); same for v.
// kv_index: nullptr => sample i uses cache slot i, else slot kv_index[i].
template <typename QT, typename KVT>
void launch_attention_rows(const QT *q, int64_t q_stride, const KVT *k, const KVT *v, int64_t kv_stride,
                           int64_t kv_sample_stride, QT *o, int64_t o_stride, int n_samples, int q_rows_per_sample,
                           int t0, int H, int dh, int mask_o, hipStream_t s);

// Single-token step: writes this step's k, v (from the fused qkv row) into the cache at position t,
// then attends keys 0..t.  qkv [B, 3W], cache [B, T, W] each for k and v, o [B, W].
template <typename AT>
void launch_decode_attention(const AT *qkv, AT *kcache, AT *vcache, AT *o, int B, int T, int t, int H, int dh,
                             int mask_o, hipStream_t s);

// Flash-style causal attention on 16-bit qkv [n_samples*T, 3W] (head size 64), o [n_samples*T, W].
template <typename HT>
void launch_flash_attention_h16(const HT *qkv, HT *o, int n_samples, int T, int H, hipStream_t s);
// the same in float32 (float32 matrix instruction), head size 64
void launch_flash_attention_f32(const float *qkv, float *o, int n_samples, int T, int H, hipStream_t s);
// on split rows, in and out (attention.hip); hs [H] and the scales of the keys as launch_head_scales leaves them
void launch_flash_attention_split(const void *qkv, void *o, const float *hs, int n_samples, int T, int H, hipStream_t s);

// Skinny 16-bit projection for single-token steps (M <= 256 rows, K % 32 == 0); same contract as
// launch_gemm_h16.
// frag: operands in the fragment-major layout of the 16x16x32 MFMA (A [M <= 64, K], Wt, and C unless
// it is a float output without residual).  Otherwise everything is row-major.
template <typename HT, typename OutT>
void launch_skinny_gemm(const HT *A, const HT *Wt, const float *bias, const float *resid, OutT *C, int M, int N, int K,
                        Epi epi, bool frag, hipStream_t s);

// The same with LayerNorm of the float32 rows Hs [M, K] fused in front (gain g, shift be); returns
// false (nothing launched) when the shape is outside what the fused kernel covers (K in
// {256, 512, 768, 1024}).  Fragment-major operands only (Hs, Wt, and a 16-bit C).
template <typename HT, typename OutT>
bool launch_skinny_ln_gemm(const float *Hs, const float *g, const float *be, const HT *Wt, const float *bias, OutT *C,
                           int M, int N, int K, Epi epi, hipStream_t s);

// Single-token attention for head size 64 with the position read from device memory (*t_dev):
// appends this step's k, v to the cache [B, T, W] and attends keys 0..t.
template <typename HT>
void launch_decode_attention_h16(const HT *qkv, HT *kcache, HT *vcache, HT *o, const int32_t *t_dev, int B, int T, int H,
                                 bool frag, hipStream_t s);

// The float32 counterparts (decode_f32.hip), everything row-major.  Projection C[M,N] = epi(LN?(A)[M,K] * Wm[K,N] + bias),
// K % 16 == 0; with g != nullptr the rows of A are normalised first (gain g, shift be; skinny_f32_ln_ok(K)).
bool skinny_f32_ln_ok(int K);
void launch_skinny_f32(const float *A, const float *g, const float *be, const float *Wm, const float *bias,
                       const float *resid, float *C, int M, int N, int K, Epi epi, hipStream_t s);
// qkv [B, 3W], caches [B, T, W], o [B, W], position *t_dev; decode_attention_f32_ok(dh)
bool decode_attention_f32_ok(int dh);
void launch_decode_attention_f32(const float *qkv, float *kcache, float *vcache, float *o, const int32_t *t_dev, int B, int T,
                                 int H, int dh, hipStream_t s);

// Step boundary of the sequential inverse: x_{t+1} from the head row of position t (eq. 5), its
// embedding into h, and t <- t+1 (device counter).  first != 0: x_0 = z_0, embedding of position 0, t <- 0.
void launch_decode_advance(const float *p, const float *z, float *x, const float *w_in, const float *b_in,
                           const float *pos, float *h, int32_t *t_dev, uint32_t *ticket, int B, int T, int D, int W,
                           int reversed, int first, bool frag, hipStream_t s);

// Jacobi epilogue.  p [n_rows, 2D] head output (row r of a sample parameterises position r+1).
// For every listed sample that is still active: x <- z*exp(alpha)+mu in place, delta, pass count,
// convergence flag.  Then the last workgroup rebuilds the active list.  shared_params != 0: p holds the head output
// of ONE sample, [T, 2D], which parameterises every listed sample (see run_jacobi: the pass from x^0 = 0).
struct JacobiState {
    float *delta;          // [B] last delta of each sample
    int32_t *iters;        // [B] passes taken
    int32_t *done;         // [B] 1 once converged or capped
    int32_t *nonfinite;    // [1] set when a sample finishes with a non-finite delta
    int32_t *active_in;    // [B] samples this pass ran on (n_listed entries)
    int32_t *active_out;   // [B] compacted list of samples still running
    uint64_t *counts;      // host memory: samples still running, and above 2^32 how many of them are marked fine (they end the list)
    uint32_t *ticket;      // [1] workgroup counter, zero before the launch, zero again after
    int32_t *fine;         // [B] 1 once a sample's delta has fallen below the refinement level (it stays 1)
};
// The update of Alg. 1 for the n samples listed in st.active_in (head output p: row block i belongs to entry i;
// with shared_params one sample's parameters serve all): x <- z * exp(alpha) + mu, delta, pass count, done flag;
// a sample whose delta falls below refine_below is marked fine.  The launches of a pass have n_listed samples together, those of
// `list`; the last workgroup of them rebuilds the list of samples that still iterate in st.active_out: first those not marked fine, then
// the fine ones, each part in increasing order, and *st.counts receives both counts.  keep_all: finished samples stay listed (first part).
void launch_jacobi_update(const float *p, const float *z, float *x, JacobiState st, int n, int T, int D, int reversed,
                          float tau, int criterion, int cap, int shared_params, float refine_below, const int32_t *list,
                          int n_listed, int keep_all, hipStream_t s);
// x^0 and state initialisation for a Jacobi block: x = 0 or z; iters = 0; done = 0; active = 0..B-1
void launch_jacobi_init(const float *z, float *x, JacobiState st, int B, int T, int D, int init, hipStream_t s);

// Sequential step epilogue: position t+1 of every sample from head row p[b, :]:
// x[b, tok(t+1), :] = z[b, tok(t+1), :] * exp(alpha) + mu.  With t = -1 copies position 0 (x_1 = y_1).
void launch_decode_epilogue(const float *p, const float *z, float *x, int B, int T, int D, int t, int reversed,
                            hipStream_t s);

// mu/alpha extraction for sjd_conditioner: shifted parameters in canonical order.
// Arguments of the persistent sequential-inverse kernel (decode_persistent.hip).  All pointers are device memory.
struct SeqLayer {
    const float *ln1_g, *ln1_b, *b_qkv, *b_o, *ln2_g, *ln2_b, *b_fc1, *b_fc2;
    const void *f_qkv, *f_o, *f_fc1, *f_fc2;  // fragment-major 16-bit weights
};
constexpr int kSeqMaxLayers = 32;
struct SeqArgs {
    SeqLayer layers[kSeqMaxLayers];  // in the kernel-argument segment: read with scalar loads, no pointer chasing
    int n_layers;
    const float *lnf_g, *lnf_b, *b_head;
    const void *f_head;
    const float *w_in, *b_in, *pos;
    const float *z;
    float *x;
    void *ws;              // activations of a step, all buffers with their slots (see decode_persistent.hip)
    void *kcache, *vcache; // [layer][max_batch][T][W] 16-bit
    size_t kv_layer_stride;  // elements between layers
    int B, T, D, reversed;
    int xpg;               // XCDs per group (1, 2, 4 or 8)
    int kv_stream;         // 1: cached rows are loaded with the streaming hint
    int kv_ahead;          // 1: the first cached rows of a pair are requested into LDS between the stages before (one row block only)
    int *sync;             // kSeqSyncWords: [0..7] members per XCD, [8] arrivals, [9] status
    int spin_max;
};
// Bytes per (row, column of width W) of the workspace: stream 4 + 3 slots of float32, qkv, attention output and MLP hidden
// (3 + 1 + 4 widths) 3 slots of 16 bits; rows for 8 groups of 16 MB.
constexpr uint32_t kSeqWsBytesPerElem = 4 * 4 + 3 * 4 + 3 * 2 * (3 + 1 + 4);
inline size_t seq_persistent_ws_bytes(int MB, int W) { return (size_t)8 * 16 * MB * W * kSeqWsBytesPerElem; }
constexpr int kSeqSyncWords = 16;
size_t seq_persistent_lds_bytes(int MB, int D);
// One workgroup of 512 threads per CU (grid = number of CUs), as a cooperative launch or a plain one.  W = 256 S.
hipError_t launch_seq_persistent(bool is_bf16, const SeqArgs &args, int MB, int S, int grid, bool cooperative,
                                 hipStream_t s);

// The sequential inverse of a narrow float32 flow's block in one launch, a workgroup per sample (decode_f32_block.hip).
struct SeqF32Layer {
    const float *ln1_g, *ln1_b, *w_qkv, *b_qkv, *w_o, *b_o, *ln2_g, *ln2_b, *w_fc1, *b_fc1, *w_fc2, *b_fc2;
};
struct SeqF32Args {
    SeqF32Layer layers[kSeqMaxLayers];
    int n_layers;
    const float *lnf_g, *lnf_b, *w_head, *b_head;   // w_head: rows head_ld floats apart, on 16-byte boundaries
    int head_ld;
    const float *w_in, *b_in, *pos, *z;
    float *x, *kcache, *vcache;                     // caches [layer][max_batch][T][W]
    size_t kv_layer_stride;
    int T, D, dh, reversed;
};
bool seq_block_f32_ok(int W, int dh, int mlp_ratio, int n_layers);
void launch_seq_block_f32(const SeqF32Args &args, int W, int B, hipStream_t s);

void launch_jacobi_trace(const float *x, const float *x_ref, JacobiState st, float *delta_out, float *err_out, int B,
                         int T, int D, hipStream_t s);
void launch_forward_epilogue(const float *p, const float *x, float *y, float *logdet, int B, int T, int D, int reversed,
                             int accumulate, hipStream_t s);
void launch_split_params(const float *p, float *mu, float *alpha, int B, int T, int D, int reversed, hipStream_t s);

// Weight preparation on the device: dst[n, k] (16-bit, row length ldb, zero padded) = src[k, n] (float [K, N]).
template <typename HT>
void launch_transpose_to_h16(const float *src, HT *dst, int K, int N, int ldb, int n_rows_padded, hipStream_t s);

// Weight preparation for the skinny kernels: fragment-major 16-bit copy of src [K, N] (see decode.hip).
template <typename HT>
void launch_weights_to_frag(const float *src, HT *dst, int K, int N, int n_rows_padded, hipStream_t s);

}  // namespace sjd

// Sequential inverse of one block (eq. 5 with the key/value cache of Sec. 3.5) of a narrow float32 flow in one launch: a workgroup
// carries one sample through all positions and layers.
//
// At widths 64 and 128 a step has next to no work in it (1.6 MB of weights at width 128 and 2 layers), and as a chain of 5 N + 2 launches
// (decode_f32.hip) it costs 3 us a link.  Inside a workgroup a link is a barrier.  What bounds it: the load path of a CU (every workgroup
// pulls the block's weights out of its L2 once per step, 6 us a layer at width 128), and the ten barriers of a layer with a trip to LDS each
// (5 us; eight waves: sixteen halve the work of each but take 29 us a step where this takes 24).  So a product's weights are requested as soon
// as the registers of the one before are free, ahead of the barriers between them, and small parameters ahead of those: loads come back in order.
// The samples share nothing: no co-residency is needed, more samples than CUs run in rounds, and a sample gives the same bits in any batch.
// Microseconds a step, per-step launches -> this: width 128, 2 layers, 4 samples of 49 tokens 45 -> 24, 256 samples 63 -> 25, 256 of 256
// tokens 70 -> 31, 4 of 1000 tokens 54 -> 36; 8 layers, 4 samples 142 -> 93; width 64, 4 layers, 32 samples 104 -> 24.
//
// A product y[n] = sum_k x[k] w[k][n]: thread (slice, group) takes four columns and an equal run of k, the partial sums of a column
// meet in LDS and are added in order of k.  Attention: W / 4 lanes hold a key of all heads (four values each, dh / 4 lanes a head), the key
// groups of a workgroup walk the cache with an online softmax each and meet once at the end.
#include "common.h"

namespace sjd {

namespace {

constexpr int SB_T = 512;        // threads

// Sums over lanes without the LDS unit, whose exchanges take a hundred clocks each: DPP inside a row of sixteen lanes, swaps across rows.
template <int CTRL> __device__ __forceinline__ float sb_dpp(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float2 sb_swap16(float x) {      // {lower, upper} row of each pair of rows
    const auto v = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return float2{__uint_as_float(v[0]), __uint_as_float(v[1])};
}
__device__ __forceinline__ float2 sb_swap32(float x) {      // {lower, upper} half of the wave
    const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return float2{__uint_as_float(v[0]), __uint_as_float(v[1])};
}
__device__ __forceinline__ float sb_sum4(float x) {         // aligned groups of 4, 8, 16, ... lanes
    x += sb_dpp<0xB1>(x);
    return x + sb_dpp<0x4E>(x);
}
__device__ __forceinline__ float sb_sum_to16(float x) { x += sb_dpp<0x141>(x); return x + sb_dpp<0x128>(x); }    // from 4 to 16
__device__ __forceinline__ float sb_add(float2 v) { return v.x + v.y; }
__device__ __forceinline__ float sb_wave_sum(float x) { return sb_add(sb_swap32(sb_add(sb_swap16(sb_sum_to16(sb_sum4(x)))))); }

// threads that share a product's column group: a power of two that divides k
constexpr int sb_slices(int K, int N) {
    int s = 1;
    while (2 * s * (N / 4) <= SB_T && K % (2 * s) == 0) s *= 2;
    return s;
}

// This thread's weights of a product: KP rows of four columns.  Loads take a matrix descriptor, one lane offset and scalar row offsets, so that
// they need one register of address.
template <int K, int N> struct SbProduct {
    static constexpr int G = N / 4, S = sb_slices(K, N), KP = K / S;
    f32x4 w[KP];
    __device__ __forceinline__ void request(const float *wm, int tid) {
        __builtin_amdgcn_sched_barrier(0);              // requested here: not earlier, where the registers are still in use, ...
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(wm), 0, K * N * 4, 0x00020000);
        asm volatile("" : "+v"(tid));
        const int s = tid / G, c = tid - s * G;
        const int off = (s * KP * N + 4 * c) * 4;       // threads past the last slice: past the matrix, zeros
#pragma unroll
        for (int i = 0; i < KP; ++i) w[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, i * N * 4, 0));
        __builtin_amdgcn_sched_barrier(0);              // ... and not where they are used
    }
    // partial sums of x (in LDS) to part[slice][N]
    __device__ __forceinline__ void partial(const float *x, float *part, int tid) {
        asm volatile("" : "+v"(tid));
        const int s = tid / G, c = tid - s * G;
        if (s >= S) return;
        f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < KP; ++i) {
            const float v = x[s * KP + i];
#pragma unroll
            for (int e = 0; e < 4; ++e) a[e] = fmaf(v, w[i][e], a[e]);
        }
        *reinterpret_cast<f32x4 *>(part + s * N + 4 * c) = a;
    }
};

// Sum of column n over S slices, in order.  Eight reads at a time: the registers hold the next product's weights meanwhile.
template <int S> __device__ __forceinline__ float sb_sum(const float *part, int N, int n) {
    float t = 0.f;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        t += part[s * N + n];
        if (s % 8 == 7) __builtin_amdgcn_sched_barrier(0);
    }
    return t;
}

// The residual stream lives in the registers of wave 0, W / 64 neighbouring columns a lane.  It takes the partial sums of a product in, and
// leaves the normalised row in LDS (biased variance, eps 1e-5).
template <int W> struct SbStream {
    static constexpr int E = W / 64;
    float h[E];
    struct Small { float bias[E], g[E], be[E]; };       // bias of the product that comes in, gain and shift of the LayerNorm behind it
    static __device__ __forceinline__ Small small(const float *__restrict__ bias, const float *__restrict__ g, const float *__restrict__ be, int lane) {
        Small p;
#pragma unroll
        for (int e = 0; e < E; ++e) { p.bias[e] = bias[lane * E + e]; p.g[e] = g[lane * E + e]; p.be[e] = be[lane * E + e]; }
        return p;
    }
    template <int S> __device__ __forceinline__ void add(const float *part, const Small &p, int lane) {
#pragma unroll
        for (int e = 0; e < E; ++e) h[e] += sb_sum<S>(part, W, lane * E + e) + p.bias[e];
    }
    __device__ __forceinline__ void normalise(const Small &p, float *xn, int lane) {
        float s = 0.f, q = 0.f;
#pragma unroll
        for (int e = 0; e < E; ++e) s += h[e];
        const float mean = sb_wave_sum(s) * (1.0f / (float)W);
#pragma unroll
        for (int e = 0; e < E; ++e) { const float d = h[e] - mean; q = fmaf(d, d, q); }
        const float rstd = 1.0f / sqrtf(sb_wave_sum(q) * (1.0f / (float)W) + 1e-5f);
#pragma unroll
        for (int e = 0; e < E; ++e) xn[lane * E + e] = (h[e] - mean) * rstd * p.g[e] + p.be[e];
    }
};

template <int W>
__global__ __launch_bounds__(SB_T) void seq_block_f32_kernel(SeqF32Args a) {
    constexpr int C = W / 4, KG = SB_T / C, NWV = SB_T / 64;   // lanes of a key, keys at a time, waves
    constexpr int U = 4;                                                    // keys in flight per thread
    __shared__ __attribute__((aligned(16))) float part[SB_T * 4];
    __shared__ __attribute__((aligned(16))) float xn[W], qkv[3 * W], o[W], ff[4 * W];
    __shared__ float wml[NWV][C][2];
    __shared__ __attribute__((aligned(16))) float wacc[NWV][W];
    extern __shared__ float dyn[];
    float *xs = dyn, *p = dyn + a.D;            // [D], [2D]
    const int T = a.T, D = a.D, LPK = a.dh / 4;
    const size_t b = blockIdx.x;
    const float scale = 1.0f / sqrtf((float)a.dh);
    const int g4 = (2 * D + 3) / 4;             // column groups of the head
    int hs = 1;                                 // and its slices
    while (2 * hs * g4 <= SB_T && 2 * hs <= W) hs *= 2;

    // the first rows of this thread's part of the embedding and head matrices stay in registers for all steps
    constexpr int ES = SB_T / W, EK = 8, HK = 4;
    const int kp = W / hs;
    float we[EK];
    f32x4 wh[HK];
#pragma unroll
    for (int i = 0; i < EK; ++i) {
        const int d = (int)threadIdx.x / W + i * ES;
        we[i] = a.w_in[(uint32_t)((d < D ? d : 0) * W + threadIdx.x % W)];
    }
    {
        const int s = (int)threadIdx.x / g4, c = (int)threadIdx.x - s * g4;
#pragma unroll
        for (int i = 0; i < HK; ++i)
            wh[i] = *reinterpret_cast<const f32x4 *>(a.w_head + (uint32_t)((s < hs && i < kp ? s * kp + i : 0) * a.head_ld + 4 * c));
    }
    SbStream<W> stream;
    constexpr int ZP = 1024 / SB_T;             // token sizes up to 1024: latent values a step ahead
    float z[ZP];
#pragma unroll
    for (int i = 0; i < ZP; ++i) {
        const int d = (int)threadIdx.x + i * SB_T;
        z[i] = d < D ? a.z[(b * T + (a.reversed ? T - 1 : 0)) * D + d] : 0.f;
    }
    for (int l = 0; l < T; ++l) {
        // copies that the optimiser cannot see through: addresses are worked out where they are used instead of being kept for all steps
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const size_t tok = a.reversed ? T - 1 - l : l;
#pragma unroll
        for (int i = 0; i < ZP; ++i) {
            const int d = tid + i * SB_T;
            if (d < D) {
                const size_t idx = (b * T + tok) * D + d;
                float v = z[i];
                if (l > 0) v = fmaf(v, expf(p[D + d]), p[d]);
                a.x[idx] = v;
                xs[d] = v;
                if (l + 1 < T) z[i] = a.z[a.reversed ? idx - D : idx + D];
            }
        }
        if (l == T - 1) break;
        __syncthreads();
        {   // embedding: D split over ES slices
            const int c = tid % W, s = tid / W;
            float t = 0.f;
#pragma unroll
            for (int i = 0; i < EK; ++i) {
                const int d = s + i * ES;
                if (d < D) t = fmaf(xs[d], we[i], t);
            }
            for (int d0 = s + EK * ES; d0 < D; d0 += 8 * ES) {      // eight loads at a time
                float w[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) w[i] = a.w_in[(uint32_t)((d0 + i * ES < D ? d0 + i * ES : d0) * W + c)];
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (d0 + i * ES < D) t = fmaf(xs[d0 + i * ES], w[i], t);
            }
            part[s * W + c] = t;
        }
        for (int ly = 0; ly < a.n_layers; ++ly) {
            const SeqF32Layer &lw = a.layers[ly];
            float *kc = a.kcache + (size_t)ly * a.kv_layer_stride + b * T * W;
            float *vc = a.vcache + (size_t)ly * a.kv_layer_stride + b * T * W;
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
            const int dc = tid % C, kg = tid / C;
            // small parameters are always requested ahead of the next product's weights: loads come back in order
            const auto p_in = SbStream<W>::small(ly == 0 ? a.b_in : a.layers[ly - 1].b_fc2, lw.ln1_g, lw.ln1_b, lane);
            if (ly == 0) {
#pragma unroll
                for (int e = 0; e < W / 64; ++e) stream.h[e] = a.pos[(size_t)l * W + lane * (W / 64) + e];
            }
            SbProduct<W, 3 * W> pq;
            pq.request(lw.w_qkv, tid);
            __syncthreads();
            if (wave == 0) {                    // what the embedding or the layer before has left in part
                if (ly == 0) stream.template add<SB_T / W>(part, p_in, lane);
                else stream.template add<SbProduct<4 * W, W>::S>(part, p_in, lane);
                stream.normalise(p_in, xn, lane);
            }
            __syncthreads();
            pq.partial(xn, part, tid);
            const float b_qkv = lw.b_qkv[tid < 3 * W ? tid : 0];
            // cached keys and values of the first U groups: they do not depend on this step
            f32x4 k4[U], v4[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {       // unconditional (a branch would wait); past the prefix a row that is there, masked below
                const int s = kg + KG * u;
                const uint32_t off = (uint32_t)((s < l ? s : l > 0 ? l - 1 : 0) * W + 4 * dc);
                k4[u] = *reinterpret_cast<const f32x4 *>(kc + off);
                v4[u] = *reinterpret_cast<const f32x4 *>(vc + off);
            }
            SbProduct<W, W> po;
            po.request(lw.w_o, tid);
            __syncthreads();
            if (tid < 3 * W) qkv[tid] = sb_sum<SbProduct<W, 3 * W>::S>(part, 3 * W, tid) + b_qkv;
            __syncthreads();
            // ---- attention of all heads; the fresh key belongs to key group 0
            const f32x4 q4 = *reinterpret_cast<const f32x4 *>(qkv + 4 * dc);
            const f32x4 kf = *reinterpret_cast<const f32x4 *>(qkv + W + 4 * dc), vf = *reinterpret_cast<const f32x4 *>(qkv + 2 * W + 4 * dc);
            if (kg == 0) {
                *reinterpret_cast<f32x4 *>(kc + (uint32_t)(l * W + 4 * dc)) = kf;
                *reinterpret_cast<f32x4 *>(vc + (uint32_t)(l * W + 4 * dc)) = vf;
            }
            auto score = [&](f32x4 k) {
                float d = fmaf(q4[3], k[3], fmaf(q4[2], k[2], fmaf(q4[1], k[1], q4[0] * k[0])));
                d = sb_sum4(d);
                if (LPK >= 8) d += sb_dpp<0x141>(d);
                if (LPK >= 16) d += sb_dpp<0x128>(d);
                if (LPK >= 32) d = sb_add(sb_swap16(d));
                return d * scale;
            };
            const float df = score(kf);
            float m = kg == 0 ? df : -INFINITY, sum = kg == 0 ? 1.f : 0.f;
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
            if (kg == 0) acc = vf;
            for (int s0 = 0; s0 < l; s0 += KG * U) {
                float d[U], mn = m;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int s = s0 + kg + KG * u;
                    if (s0 > 0) {
                        const uint32_t off = (uint32_t)((s < l ? s : l - 1) * W + 4 * dc);
                        k4[u] = *reinterpret_cast<const f32x4 *>(kc + off);
                        v4[u] = *reinterpret_cast<const f32x4 *>(vc + off);
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    d[u] = score(k4[u]);
                    if (s0 + kg + KG * u >= l) d[u] = -INFINITY;
                    mn = fmaxf(mn, d[u]);
                }
                const float mu = mn == -INFINITY ? 0.f : mn;
                const float corr = expf(m - mu);
                m = mn;
                sum *= corr;
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] *= corr;
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const float pr = expf(d[u] - mu);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[e] = fmaf(pr, v4[u][e], acc[e]);
                    sum += pr;
                }
            }
            // the key groups of a wave, then the waves in order
            float mw = m;
            if (C == 16) { const float2 v = sb_swap16(mw); mw = fmaxf(v.x, v.y); }
            { const float2 v = sb_swap32(mw); mw = fmaxf(v.x, v.y); }
            const float f = expf(m - (mw == -INFINITY ? 0.f : mw));
            auto over_groups = [&](float x) {
                x *= f;
                if (C == 16) x = sb_add(sb_swap16(x));
                return sb_add(sb_swap32(x));
            };
            sum = over_groups(sum);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = over_groups(acc[e]);
            if (lane < C) {
                wml[wave][dc][0] = mw; wml[wave][dc][1] = sum;
                *reinterpret_cast<f32x4 *>(&wacc[wave][4 * dc]) = acc;
            }
            __syncthreads();
            if (tid < W) {
                const int c = tid >> 2;
                float mm = wml[0][c][0], den = 0.f, num = 0.f;
#pragma unroll
                for (int w = 1; w < NWV; ++w) mm = fmaxf(mm, wml[w][c][0]);
#pragma unroll
                for (int w = 0; w < NWV; ++w) {
                    const float fw = expf(wml[w][c][0] - mm);
                    den = fmaf(wml[w][c][1], fw, den);
                    num = fmaf(wacc[w][tid], fw, num);
                }
                o[tid] = num / den;
            }
            __syncthreads();
            po.partial(o, part, tid);
            const auto p_mid = SbStream<W>::small(lw.b_o, lw.ln2_g, lw.ln2_b, lane);
            SbProduct<W, 4 * W> p1;
            p1.request(lw.w_fc1, tid);
            __syncthreads();
            if (wave == 0) {
                stream.template add<SbProduct<W, W>::S>(part, p_mid, lane);
                stream.normalise(p_mid, xn, lane);
            }
            __syncthreads();
            p1.partial(xn, part, tid);
            const float b_fc1 = lw.b_fc1[tid < 4 * W ? tid : 0];
            SbProduct<4 * W, W> p2;
            p2.request(lw.w_fc2, tid);
            __syncthreads();
            if (tid < 4 * W) ff[tid] = gelu_erf(sb_sum<SbProduct<W, 4 * W>::S>(part, 4 * W, tid) + b_fc1);
            __syncthreads();
            p2.partial(ff, part, tid);
        }
        const auto p_end = SbStream<W>::small(a.layers[a.n_layers - 1].b_fc2, a.lnf_g, a.lnf_b, lane);
        __syncthreads();
        if (wave == 0) {
            stream.template add<SbProduct<4 * W, W>::S>(part, p_end, lane);
            stream.normalise(p_end, xn, lane);
        }
        __syncthreads();
        // ---- head: [mu | alpha] of position l + 1
        {
            const int s = tid / g4, c = tid - s * g4;
            if (s < hs) {
                f32x4 t = {0.f, 0.f, 0.f, 0.f};
                auto take = [&](int k, f32x4 w) {
                    const float v = xn[k];
#pragma unroll
                    for (int e = 0; e < 4; ++e) t[e] = fmaf(v, w[e], t[e]);
                };
#pragma unroll
                for (int i = 0; i < HK; ++i)
                    if (i < kp) take(s * kp + i, wh[i]);
                for (int k0 = HK; k0 < kp; k0 += HK) {              // kp is a power of two, HK loads at a time
                    f32x4 w[HK];
#pragma unroll
                    for (int i = 0; i < HK; ++i) w[i] = *reinterpret_cast<const f32x4 *>(a.w_head + (uint32_t)((s * kp + k0 + i) * a.head_ld + 4 * c));
#pragma unroll
                    for (int i = 0; i < HK; ++i) take(s * kp + k0 + i, w[i]);
                }
                *reinterpret_cast<f32x4 *>(part + (s * g4 + c) * 4) = t;
            }
        }
        __syncthreads();
        for (int n = tid; n < 2 * D; n += SB_T) {
            float t = part[n];
            for (int s = 1; s < hs; ++s) t += part[s * g4 * 4 + n];
            p[n] = t + a.b_head[n];
        }
        __syncthreads();
    }
}

}  // namespace

bool seq_block_f32_ok(int W, int dh, int mlp_ratio, int n_layers) {
    return (W == 64 || W == 128) && (dh == 16 || dh == 32 || dh == 64 || dh == 128) && mlp_ratio == 4 && n_layers <= kSeqMaxLayers;
}

void launch_seq_block_f32(const SeqF32Args &args, int W, int B, hipStream_t s) {
    const size_t lds = (size_t)3 * args.D * sizeof(float);
    if (W == 128) hipLaunchKernelGGL(seq_block_f32_kernel<128>, dim3(B), dim3(SB_T), lds, s, args);
    else hipLaunchKernelGGL(seq_block_f32_kernel<64>, dim3(B), dim3(SB_T), lds, s, args);
}

}  // namespace sjd

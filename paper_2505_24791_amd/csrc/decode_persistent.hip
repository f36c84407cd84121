// Sequential inverse of one block (eq. 5 with the key/value cache of Sec. 3.5) as ONE persistent
// kernel, for the 16-bit modes with head size 64.
//
// A step of the sequential inverse is a chain of 5 N dependent skinny products on a handful of rows; launched
// one by one every link costs a kernel boundary plus a cold start.  Here the chain runs inside one cooperative
// launch of one workgroup per CU.  The workgroups of `xpg` neighbouring XCDs (1, 2, 4 or 8; seq_groups.h) form a group; each
// group takes an equal share of the samples and carries them through the whole block on its own.  Inside a group
// every product is split by output columns over the members, attention by (sample, head) pairs.
//
// What bounds it is the latency of a link: what one member writes all others need next.  There is no barrier: a
// buffer is filled with a word that no result has (kEmpty, a NaN pattern) before it is used, and a reader simply
// loads its operands again until no word of them is empty.  Every 32-bit word is its own flag, so the order in
// which words arrive does not matter.  Loads carry the sc1 scope bit (agent scope).  So do the stores of a group of several XCDs, which is coherent
// between XCDs: past the L2 of either side, to the memory behind it and back (an all-gather of 2 to 64 KB, a round of a loop of nothing else: 2.2 to 2.8 us
// among 64 to 256 workgroups); a group of one XCD stores to its L2, and the loads find the words there (kStoreBits).  Microseconds a step of
// one-XCD groups, stores of agent scope -> to the L2: width 256, 6 layers, 37 samples 77.5 -> 57.1; 4 layers, 128 samples 70.6 -> 44.6; width 512, 4 layers, 64 samples
// 81.1 -> 67.6, 128 97.0 -> 84.8; width 768, 8 layers, 256 samples 422 -> 396; width 1024, 4 layers, 200 samples 260 -> 251.
//
// Life of a buffer.  Results rotate through three slots (the residual stream after the MLP and the embedding: four).
// A member that has written slot q of a buffer empties what it had written in slot q-1 (stream: q-2), and every
// store is acknowledged before the member's next write.  That is safe because a member writes use q of a stage only
// after the complete input of that use has arrived, which depends on every member that read use q-1 having finished
// (all of a stage's outputs are needed by the next, and so on round the chain); and because a reader gets to use
// q+2 (whose slot was emptied at q) only after it has seen, directly or through others, use q+1, which was written
// after the emptying had been acknowledged.  The last stream of a step is read by every member (the head), which is
// why the stream keeps one slot more: use q is written by the next step's MLP output at the earliest, when all
// members have shown results that come after their head.  Every wait is bounded: after spin_max attempts a workgroup
// records an error, stops waiting and leaves at the end of the step, so do the others in turn, and the host reports the failure.
//
// The arithmetic per row: LayerNorm statistics per slice of 1/8 of a row (mean, then centred sum of squares), slices
// combined by the parallel formula for variances; 16x16x32 MFMA with K split over the 8 waves of a workgroup and partial sums
// added in wave order; float32 residual stream.  A row's result does not depend on which group or member computes it.
#include "common.h"
#include "seq_groups.h"
#include <type_traits>

namespace sjd {

namespace {

constexpr int P_NW = 8;  // waves per workgroup
constexpr int P_THREADS = 64 * P_NW;
constexpr int P_EB = 2;  // embedding units of a member whose w_in slice is kept in LDS
constexpr uint32_t kEmpty = 0xFFFFFFFFu;
constexpr uint32_t kNowhere = 0xFFFFFFF0u;   // beyond every buffer: a load there returns zeros without any traffic

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

__device__ __forceinline__ rsrc_t make_rsrc(const void *p, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
// 16-byte loads of exchanged words and of cached rows, at agent scope (bit 4, sc1): never served by this CU's vector cache, so each attempt of
// a wait sees what the L2 has.
__device__ __forceinline__ i32x4 ld16(rsrc_t rs, uint32_t byte_off) {
    return __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)byte_off, 0, 16));
}
// Stores of exchanged words.  ONE: the group is one XCD, all of whose CUs share an L2; the vector cache writes through to it, so a plain store
// is there once it is acknowledged, and loads that pass by the vector cache find it (a wave's own would have to).  Else agent scope.
template <bool ONE> constexpr int kStoreBits = ONE ? 0 : 16;
// the same for rows of a key/value cache too large for the memory-side cache, with the streaming hint on top: a row is read once per
// step and should not displace the weights, which every step reads again
__device__ __forceinline__ i32x4 ld16_stream(rsrc_t rs, uint32_t byte_off) {
    return __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)byte_off, 0, 16 | 2));
}
// `off` where the lane has something to read, else kNowhere: a select that the compiler must not turn into a branch with a
// load (and a wait) on either side
__device__ __forceinline__ uint32_t where(bool live, uint32_t off) {
    uint32_t r = live ? off : kNowhere;
    asm("" : "+v"(r));
    return r;
}
// Sums over lanes without the LDS unit: within a row of sixteen lanes by DPP, across rows by the swap instructions.
template <int CTRL> __device__ __forceinline__ float dpp(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float sum8(float x) {       // lanes that agree in bits 3..5
    x += dpp<0xB1>(x);                                  // lane ^ 1
    x += dpp<0x4E>(x);                                  // lane ^ 2
    return x + dpp<0x141>(x);                           // mirrored within eight: the other half of them
}
__device__ __forceinline__ float sum_rows(float x) {   // lanes that agree in bits 0..3
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
// a lane of the lower half gets a's sum over both halves, one of the upper half b's; the same for even and odd rows of sixteen
__device__ __forceinline__ float add_halves32(float a, float b) {
    const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(v[0]) + __uint_as_float(v[1]);
}
__device__ __forceinline__ float add_halves16(float a, float b) {
    const auto v = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(v[0]) + __uint_as_float(v[1]);
}
__device__ __forceinline__ float max_rows(float x) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
// A result must not look empty: the one NaN pattern becomes another NaN.
__device__ __forceinline__ int flagged(float v) {
    const uint32_t w = __float_as_uint(v);
    return (int)(w == kEmpty ? 0x7FC00000u : w);
}
__device__ __forceinline__ int flagged(int two_halves) { return two_halves == -1 ? 0x7FFF7FFF : two_halves; }
template <bool ONE> __device__ __forceinline__ void st16(rsrc_t rs, uint32_t byte_off, i32x4 v) { __builtin_amdgcn_raw_buffer_store_b128(v, rs, (int)byte_off, 0, kStoreBits<ONE>); }
template <bool ONE> __device__ __forceinline__ void st8(rsrc_t rs, uint32_t byte_off, i32x2 v) { __builtin_amdgcn_raw_buffer_store_b64(v, rs, (int)byte_off, 0, kStoreBits<ONE>); }
template <bool ONE> __device__ __forceinline__ void st4(rsrc_t rs, uint32_t byte_off, int v) { __builtin_amdgcn_raw_buffer_store_b32(v, rs, (int)byte_off, 0, kStoreBits<ONE>); }

typedef __attribute__((address_space(3))) int LdsInt;   // LDS, not the generic address space: no flat accesses

struct Ctx {
    int tid, lane, wave, r, kg;
    int slot, n;        // this workgroup's index in its group, members of the group
    int rb0;            // first 16-row block of the group in the workspaces
    int row0, nrows;    // first sample of the group, samples of the group
    int cw;             // columns of a unit of the residual projections (4, 8 or 16)
    int spin_max;
    bool kv_stream;     // cached rows are loaded with the streaming hint
    int *status;
    LdsInt *bad;        // a wait of this workgroup gave up
};

// A copy of the per-thread indices that the optimiser cannot see through: addresses derived from it
// are recomputed where they are used instead of being hoisted out of the step loop and kept in
// registers for the whole kernel (which costs far more than the few integer instructions).
__device__ __forceinline__ Ctx local_ctx(const Ctx &c) {
    Ctx d = c;
    asm volatile("" : "+v"(d.lane), "+v"(d.tid), "+v"(d.r), "+v"(d.kg));
    d.wave = __builtin_amdgcn_readfirstlane(d.wave);
    d.slot = __builtin_amdgcn_readfirstlane(d.slot);
    d.rb0 = __builtin_amdgcn_readfirstlane(d.rb0);
    asm volatile("" : "+s"(d.wave), "+s"(d.slot), "+s"(d.rb0));
    return d;
}

// Load N pieces of 16 bytes until no word of them is empty.  Afterwards everything this wave has stored or requested so
// far is complete (the wait is free: the operands requested before the poll are needed next).  Reloading only the pieces that
// were missing, or pausing between attempts, was slower or made no difference.
template <int N, class OFF>
__device__ __forceinline__ void poll16(const Ctx &c, rsrc_t rs, OFF off, i32x4 (&v)[N]) {
    int it = 0;
    while (true) {
        asm volatile("" ::: "memory");
#pragma unroll
        for (int u = 0; u < N; ++u) v[u] = ld16(rs, off(u));
        uint32_t m = 0;
#pragma unroll
        for (int u = 0; u < N; ++u)
            m = max(m, max(max((uint32_t)v[u].x, (uint32_t)v[u].y), max((uint32_t)v[u].z, (uint32_t)v[u].w)));
        if (__builtin_amdgcn_ballot_w64(m == kEmpty) == 0) break;
        if (++it > c.spin_max || ((it & 63) == 0 && *c.bad)) {   // after one wait of the workgroup gave up the others do not start
            if (c.lane == 0) {
                *c.bad = 1;
                __hip_atomic_store(c.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            break;
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
}

// A member without a share of a stage still requests its part of the cached rows: behind the same wait and barrier as in the stage.
template <class AHEAD> __device__ __forceinline__ void idle_ahead(AHEAD ahead) {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
    ahead();
}

// C[:, blocks of this member] = epi(LayerNorm(stream) * Wt^T + bias) for the group's rows, K = W = 256 S.  The stream
// (at in_off) is float32 fragment-major, Wt fragment-major; 16-column block cb belongs to member cb % n, CB blocks a round.  Weights are the first
// matrix operand and rows the second, so a lane ends up with four consecutive columns of one row.
// 16-bit results go to out_off (fragment-major; the member's part at empty_off is emptied); with LOCAL the float32
// result goes to the workgroup's own buffer (row-major [16 MB][N], row 0 = the group's first row) and the member takes every block.
template <typename HT, int MB, int S, int CB, int EPI, bool LOCAL, bool ONE, class AHEAD>
__device__ __forceinline__ void ln_gemm_stage(const Ctx &c_in, rsrc_t ws, uint32_t in_off, const float *__restrict__ g,
                                              const float *__restrict__ be, const HT *__restrict__ Wt,
                                              const float *__restrict__ bias, uint32_t out_off, uint32_t empty_off,
                                              float *local, int N, f32x4v *red, float2 *stat, AHEAD ahead) {
    typedef typename Half16<HT>::v8 v8;
    typedef typename Half16<HT>::v4 v4;
    constexpr int W = 256 * S, KS = 8 * S;
    const int nbt = (N + 15) >> 4;
    const int slot = LOCAL ? 0 : c_in.slot, n = LOCAL ? 1 : c_in.n;
    if (slot >= nbt) { idle_ahead(ahead); return; }
    const Ctx c = local_ctx(c_in);
    const int k0 = c.wave * 32 * S + c.kg * 8;
    v8 w[CB][S];
    auto fetch = [&](int cb0) {     // clamped, so that the loads are unconditional; blocks past the end are never used
#pragma unroll
        for (int cc = 0; cc < CB; ++cc) {
            int cb = cb0 + cc * n;
            cb = cb < nbt ? cb : nbt - 1;
#pragma unroll
            for (int s = 0; s < S; ++s)
                w[cc][s] = *reinterpret_cast<const v8 *>(Wt + (((size_t)cb * KS + c.wave * S + s) * 64 + c.lane) * 8);
        }
    };
    fetch(slot);
    f32x4 gr[S][2], br[S][2];
#pragma unroll
    for (int s = 0; s < S; ++s) {
        gr[s][0] = *reinterpret_cast<const f32x4 *>(g + k0 + 32 * s);
        gr[s][1] = *reinterpret_cast<const f32x4 *>(g + k0 + 32 * s + 4);
        br[s][0] = *reinterpret_cast<const f32x4 *>(be + k0 + 32 * s);
        br[s][1] = *reinterpret_cast<const f32x4 *>(be + k0 + 32 * s + 4);
    }
    constexpr int NQ = (CB * MB + P_NW - 1) / P_NW;   // output blocks a wave finishes in a round (q = wave, wave + 8, ...)
    float bv[NQ][4];
    const rsrc_t bias_rs = make_rsrc(bias, (uint32_t)N * 4u);
    auto fetch_bias = [&](int cb0) {
#pragma unroll
        for (int qi = 0; qi < NQ; ++qi) {
            const int q = c.wave + qi * P_NW;
            const int col = (cb0 + (q / MB) * n) * 16 + 4 * c.kg;
#pragma unroll
            for (int v = 0; v < 4; ++v)     // zeros past the end
                bv[qi][v] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(bias_rs, (int)(col + v) * 4, 0, 0));
        }
    };
    fetch_bias(slot);
    __builtin_amdgcn_sched_barrier(0);
    i32x4 raw[MB * S * 2];
    poll16(c, ws, [&](int u) {
        const int i = u / (2 * S), s = (u >> 1) % S;
        const uint32_t off = in_off + (uint32_t)((((c.rb0 + i) * KS + c.wave * S + s) * 64 + c.lane) * 8) * 4u + (u & 1) * 16u;
        return where(i * 16 + c.r < c.nrows, off);
    }, raw);
    auto x = [&](int i, int s, int h2, int e) { return __int_as_float(raw[(i * S + s) * 2 + h2][e]); };
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        float sum = 0.f;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) sum += x(i, s, 0, e) + x(i, s, 1, e);
        sum = sum_rows(sum);
        const float mw = sum * (1.0f / (32.f * S));
        float m2 = 0.f;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
                for (int e = 0; e < 4; ++e) { const float d = x(i, s, h2, e) - mw; m2 = fmaf(d, d, m2); }
        m2 = sum_rows(m2);
        if (c.kg == 0) stat[c.wave * (MB * 16) + i * 16 + c.r] = float2{mw, m2};
    }
    __syncthreads();
    ahead();
    v8 fa[MB][S];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        float2 st[P_NW];
        float mean = 0.f;
#pragma unroll
        for (int q = 0; q < P_NW; ++q) { st[q] = stat[q * (MB * 16) + i * 16 + c.r]; mean += st[q].x; }
        mean *= 1.0f / P_NW;
        float between = 0.f, within = 0.f;
#pragma unroll
        for (int q = 0; q < P_NW; ++q) { const float d = st[q].x - mean; between = fmaf(d, d, between); within += st[q].y; }
        const float rstd = 1.0f / sqrtf(fmaf(32.f * S, between, within) * (1.0f / (float)W) + 1e-5f);
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    fa[i][s][4 * h2 + e] = from_f32<HT>((x(i, s, h2, e) - mean) * rstd * gr[s][h2][e] + br[s][h2][e]);
    }
    for (int cb0 = slot; cb0 < nbt; cb0 += CB * n) {
        if (cb0 != slot) {
            __syncthreads();   // the previous round's partial sums have been read
            fetch(cb0);
            fetch_bias(cb0);
            __builtin_amdgcn_s_waitcnt(0x0F70);   // they are needed next; and no load is left under way behind the results' stores
        }
#pragma unroll
        for (int cc = 0; cc < CB; ++cc)
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                f32x4v acc = f32x4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < S; ++s) acc = Mfma16<HT>::run(w[cc][s], fa[i][s], acc);
                red[(c.wave * (CB * MB) + cc * MB + i) * 64 + c.lane] = acc;
            }
        __syncthreads();
        // output block q = (cc, i) is summed in wave order and finished by wave q % 8
#pragma unroll
        for (int qi = 0; qi < NQ; ++qi) {
            const int q = c.wave + qi * P_NW;
            if (q >= CB * MB) break;
            const int cc = q / MB, i = q % MB;
            const int cb = cb0 + cc * n;
            if (cb >= nbt) continue;
            f32x4v t = red[q * 64 + c.lane];
#pragma unroll
            for (int p = 1; p < P_NW; ++p) t += red[(p * (CB * MB) + q) * 64 + c.lane];
            const int row = i * 16 + c.r, col = cb * 16 + 4 * c.kg;
            if constexpr (LOCAL) {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (col + v < N) local[row * N + col + v] = t[v] + bv[qi][v];
            } else {
                v4 h;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float val = t[v] + bv[qi][v];
                    if (EPI == EPI_BIAS_GELU) val = gelu_erf_h16(val);
                    h[v] = from_f32<HT>(val);
                }
                if (row < c.nrows) {
                    const i32x2 two = __builtin_bit_cast(i32x2, h);
                    const uint32_t eo = (uint32_t)frag_off(c.rb0 * 16 + row, col, N >> 5) * 2u;
                    st8<ONE>(ws, out_off + eo, i32x2{flagged(two.x), flagged(two.y)});
                    st8<ONE>(ws, empty_off + eo, i32x2{-1, -1});
                }
            }
        }
    }
}

// stream_out[:, units of this member] = stream_in + A * Wt^T + bias for the group's rows; N = W = 256 S, K = KMUL * W.
// A (at a_off) 16-bit fragment-major, the streams float32 fragment-major.  A unit is cw columns: with many members a 16-column
// block is shared out among two or four of them (the lanes of the other columns repeat theirs), so that every
// member pulls an equal, small piece of the weights; unit u belongs to member u % n.
template <typename HT, int MB, int S, int KMUL, bool ONE, class AHEAD>
__device__ __forceinline__ void gemm_resid_stage(const Ctx &c_in, rsrc_t ws, uint32_t a_off, const HT *__restrict__ Wt,
                                                 const float *__restrict__ bias, uint32_t in_off, uint32_t out_off,
                                                 uint32_t empty_off, f32x4v *red, AHEAD ahead) {
    typedef typename Half16<HT>::v8 v8;
    constexpr int W = 256 * S, KSN = W / 32, KSA = 8 * S * KMUL, KSW = S * KMUL;
    const int nu = W / c_in.cw;
    if (c_in.slot >= nu) { idle_ahead(ahead); return; }
    const Ctx c = local_ctx(c_in);
    const int cmask = c.cw - 1;
    v8 w[KSW];
    float bv[4];
    uint32_t eo;                                // this lane's four columns of a stream row (wave i < MB: row block i)
    auto fetch = [&](int u) {
        const int col0 = u * c.cw, cb = col0 >> 4, cl = (col0 & 15) + (c.r & cmask);
#pragma unroll
        for (int k = 0; k < KSW; ++k)
            w[k] = *reinterpret_cast<const v8 *>(Wt + (((size_t)cb * KSA + c.wave * KSW + k) * 64 + c.kg * 16 + cl) * 8);
        const int col = col0 + ((4 * c.kg) & cmask);
#pragma unroll
        for (int v = 0; v < 4; ++v) bv[v] = bias[col + v];
        eo = (uint32_t)frag_off((c.rb0 + c.wave) * 16 + c.r, col, KSN) * 4u;
    };
    const bool finish = c.wave < MB && c.wave * 16 + c.r < c.nrows && 4 * c.kg < c.cw;
    fetch(c.slot);
    __builtin_amdgcn_sched_barrier(0);
    i32x4 raw[MB * KSW + 1];                    // the activation, and the stream values of the first unit
    poll16(c, ws, [&](int u) {
        if (u == MB * KSW) return where(finish, in_off + eo);
        const int i = u / KSW, k = u % KSW;
        const uint32_t off = a_off + (uint32_t)((((c.rb0 + i) * KSA + c.wave * KSW + k) * 64 + c.lane) * 8) * 2u;
        return where(i * 16 + c.r < c.nrows, off);
    }, raw);
    i32x4 rv[1] = {raw[MB * KSW]};
    for (int u = c.slot; u < nu; u += c.n) {
        if (u != c.slot) {
            __syncthreads();                    // the previous unit's partial sums have been read
            fetch(u);
            poll16(c, ws, [&](int) { return where(finish, in_off + eo); }, rv);
        }
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            f32x4v acc = f32x4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < KSW; ++k) acc = Mfma16<HT>::run(w[k], __builtin_bit_cast(v8, raw[i * KSW + k]), acc);
            red[(c.wave * MB + i) * 64 + c.lane] = acc;
        }
        __syncthreads();
        if (u == c.slot) ahead();
        if (finish) {
            f32x4v t = red[c.wave * 64 + c.lane];
#pragma unroll
            for (int p = 1; p < P_NW; ++p) t += red[(p * MB + c.wave) * 64 + c.lane];
            i32x4 out;
#pragma unroll
            for (int v = 0; v < 4; ++v) out[v] = flagged((t[v] + bv[v]) + __int_as_float(rv[0][v]));
            st16<ONE>(ws, out_off + eo, out);
            st16<ONE>(ws, empty_off + eo, i32x4{-1, -1, -1, -1});
        }
    }
}

// Single-token attention of the group's (sample, head) pairs against the cache at position t: pair (row, h) belongs to
// member (row * H + h) % n, which also appends this step's k and v to the cache.  A pair is handled by four waves: 32
// key groups x 8 sixteen-byte chunks of the head, two pairs at a time per workgroup.  A key group walks its keys in
// batches of P_AU with an online softmax of its own; the groups meet once, at the end (the wave's eight by lane
// exchange, the four waves through LDS).  The partition of the keys and the order of the sums depend on t only.
// Cached rows do not depend on the current step: the first batch is requested before the poll for q, k, v, and each
// next batch (of this pair or the next) as soon as the registers of the current one have been used.
// What bounds it: memory and the load path of a CU (64 bytes a clock) where the prefix is long, else the serial chain behind the last
// score: groups hand on the half of their sums that they do not keep, and a wave finishes a pair, one element a lane.  Microseconds a step, with
// eight lanes finishing 64 elements, three exchanges a sum and loads issued for rows past the prefix -> now: width 512, 4 layers, one sample 57.5 ->
// 55.6; width 256, 6 layers, 37 samples 81.5 -> 77.5; width 768, 8 layers, 256 samples 445 -> 420; width 1024, 8 layers, 32 samples of
// 1024 tokens 282 -> 270.
//
// AHEAD: the first 32 P_LU keys of a member's first two pairs come out of LDS: while the other four stages of a layer exchange
// their results the memory that holds the cache is idle, and what it costs to stream the cached rows of a long prefix is its bandwidth.
// They are requested by LDS-direct loads between those stages (kv_ahead), each thread the pieces that it reads itself, so the order
// "requested, waited for by the next poll, read" needs no barrier.  The registers then hold the P_AU rows that follow: batch 0 is
// rows 0..P_LU-1 from LDS and the others from registers, and the first P_LU registers are a batch further.
// Same bits.  Microseconds a step without -> with: width 1024, 8 layers, 19 samples of 777 tokens 225 -> 216, 32 of 1024 270 -> 258.
constexpr int P_NSUB = 2;
constexpr int P_AU = 8;  // cache rows per thread and batch
constexpr int P_LU = 5;  // of batch 0 of the first pairs: rows in LDS (what it has left of 160 KB at token size 64)
constexpr int P_AHEAD_BYTES = 2 * P_LU * P_THREADS * 16;
constexpr int P_AHEAD_STEPS[5] = {0, 3, 5, 8, 10};   // loads per thread after each of the four stages: K rows 0..P_LU-1, then V rows
static_assert(P_AHEAD_STEPS[4] == 2 * P_LU, "every row is requested");

// Part `part` (0..3) of the rows that the attention of a layer finds in LDS, for position t.  A row is requested at the
// earliest behind the barrier of the stage that follows the attention which wrote it, and the writer has waited for its store by then.
template <int S>
__device__ __forceinline__ void kv_ahead(const Ctx &c_in, int part, const void *kc, const void *vc, int t, int T, uint32_t lds0) {
    constexpr int W = 256 * S, H = W / 64;
    const Ctx c = local_ctx(c_in);
    const int sub = c.wave >> 2, stid = c.tid & 255, dc = stid & 7, sg = stid >> 3;
    const int pi = c.slot + sub * c.n;
    if (t <= 0 || pi >= c.nrows * H) return;
    const int row = pi / H, h = pi - row * H;
    const uint32_t base = (uint32_t)(((size_t)(c.row0 + row) * T) * W + h * 64 + dc * 8) * 2u;
#pragma unroll
    for (int i = 0; i < 2 * P_LU; ++i) {
        if (i < P_AHEAD_STEPS[part] || i >= P_AHEAD_STEPS[part + 1]) continue;
        const int u = i < P_LU ? i : i - P_LU;
        if (32 * u >= t) continue;
        const int s = sg + 32 * u;
        const uint32_t off = base + (uint32_t)(s < t ? s : t - 1) * (W * 2u);    // past the end: a row that is there, its score is masked
        const uint32_t dst = lds0 + (uint32_t)(i * P_THREADS + c.wave * 64) * 16u;
        const void *src = i < P_LU ? kc : vc;
        // 64 lanes x 16 bytes from (scalar base + lane offset) to 1 KB of LDS at M0, past this CU's vector cache; nothing else here uses M0
        if (c.kv_stream)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 sc1 nt" :: "s"(dst), "v"(off), "s"(src) : "memory");
        else
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 sc1" :: "s"(dst), "v"(off), "s"(src) : "memory");
    }
}

template <typename HT, int MB, int S, bool AHEAD, bool ONE>
__device__ __forceinline__ void attention_stage(const Ctx &c_in, rsrc_t ws, uint32_t qkv_off, HT *kc, HT *vc, rsrc_t kc_rs,
                                                rsrc_t vc_rs, uint32_t out_off, uint32_t empty_off, int t, int T,
                                                float *opart, float2 *wst, int &par, const i32x4 *ahead) {
    typedef typename Half16<HT>::v8 v8;
    constexpr int W = 256 * S, H = W / 64, KS3 = 3 * W / 32;
    const int npairs = c_in.nrows * H;
    if (c_in.slot >= npairs) return;
    const Ctx c = local_ctx(c_in);
    const int sub = c.tid >> 8, stid = c.tid & 255;
    const int dc = stid & 7, sg = stid >> 3;               // chunk of the head, key group (0..31)
    const int mine = (npairs - c.slot + c.n - 1) / c.n;    // pairs of this member
    const int nb = (t + 32 * P_AU - 1) / (32 * P_AU);      // batches of cached keys
    auto pair_of = [&](int k0) { return c.slot + (k0 + sub) * c.n; };
    auto rows = [&](rsrc_t rs, int k0, int jb, int u0, int u1, i32x4 (&v)[P_AU]) {   // rows u0 <= u < u1 of batch jb
        const bool valid = k0 + sub < mine;
        const int pi = valid ? pair_of(k0) : 0, row = pi / H, h = pi - row * H;
        const uint32_t base = (uint32_t)(((size_t)(c.row0 + row) * T) * W + h * 64 + dc * 8) * 2u;
        auto all = [&](auto load) {
#pragma unroll
            for (int u = 0; u < P_AU; ++u) {
                if (u < u0 || u >= u1) continue;
                const int s0 = 32 * (jb * P_AU + u), s = s0 + sg;
                // a load takes its time at the cache also where there is nothing to read
                if (s0 < t) v[u] = load(rs, where(valid && s < t, base + (uint32_t)s * (W * 2u))); else v[u] = i32x4{0, 0, 0, 0};
            }
        };
        if (c.kv_stream) all([](rsrc_t r, uint32_t off) { return ld16_stream(r, off); });
        else all([](rsrc_t r, uint32_t off) { return ld16(r, off); });
    };
    i32x4 kk[P_AU], vv[P_AU];
    if (nb > 0) {
        if constexpr (AHEAD) {
            rows(kc_rs, 0, 0, P_LU, P_AU, kk); rows(vc_rs, 0, 0, P_LU, P_AU, vv);
            rows(kc_rs, 0, 1, 0, P_LU, kk); rows(vc_rs, 0, 1, 0, P_LU, vv);
        } else { rows(kc_rs, 0, 0, 0, P_AU, kk); rows(vc_rs, 0, 0, 0, P_AU, vv); }
    }
    __builtin_amdgcn_sched_barrier(0);
    for (int k0 = 0; k0 < mine; k0 += P_NSUB) {
        const bool valid = (k0 + sub) < mine;
        const int pi = valid ? pair_of(k0) : 0;
        const int row = pi / H, h = pi - row * H;
        const int wsrow = c.rb0 * 16 + row;
        i32x4 fresh[3];
        poll16(c, ws, [&](int part) {
            return where(valid, qkv_off + (uint32_t)frag_off(wsrow, part * W + h * 64 + dc * 8, KS3) * 2u);
        }, fresh);
        const v8 q8 = __builtin_bit_cast(v8, fresh[0]), kf = __builtin_bit_cast(v8, fresh[1]), vf = __builtin_bit_cast(v8, fresh[2]);
        if (valid && stid < 16) {   // threads 0..7 hold the fresh k chunks, 8..15 the fresh v chunks (dc = stid & 7)
            HT *dst = (stid < 8 ? kc : vc) + ((size_t)(c.row0 + row) * T + t) * W + h * 64 + dc * 8;
            *reinterpret_cast<v8 *>(dst) = stid < 8 ? kf : vf;
        }
        // softmax scale 1/sqrt(64) and log2(e) in one factor: the probabilities are powers of two
        auto score = [&](v8 k8) { return sum8(Half16<HT>::dot(q8, k8)) * (0.125f * 1.44269504088896340736f); };
        // the fresh key belongs to key group 0
        const float df = score(kf);
        float m = sg == 0 ? df : -INFINITY, l = sg == 0 ? 1.f : 0.f, acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = sg == 0 ? (float)vf[e] : 0.f;
        auto batch = [&](auto from_lds, int jb) {
            constexpr int LU = decltype(from_lds)::value ? P_LU : 0;
            const bool more = jb + 1 < nb;
            const int nk0 = more ? k0 : k0 + P_NSUB, njb = more ? jb + 1 : 0;
            const bool next = more || nk0 < mine;
            float d[P_AU], mn = m;
#pragma unroll
            for (int u = 0; u < P_AU; ++u) {
                d[u] = score(__builtin_bit_cast(v8, u < LU ? ahead[u * P_THREADS + c.tid] : kk[u]));
                if (sg + 32 * (jb * P_AU + u) >= t) d[u] = -INFINITY;
                mn = fmaxf(mn, d[u]);
            }
            if (next) { if (LU && more) rows(kc_rs, nk0, njb, P_LU, P_AU, kk); else rows(kc_rs, nk0, njb, 0, P_AU, kk); }
            const float mu = mn == -INFINITY ? 0.f : mn;       // a key group may not have any key yet
            const float corr = __builtin_amdgcn_exp2f(m - mu);
            m = mn;
            l *= corr;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] *= corr;
#pragma unroll
            for (int u = 0; u < P_AU; ++u) {
                const float p = __builtin_amdgcn_exp2f(d[u] - mu);
                i32x4 vr = vv[u];
                if (u < LU) { if (32 * u < t) vr = ahead[(P_LU + u) * P_THREADS + c.tid]; else vr = i32x4{0, 0, 0, 0}; }   // not requested: LDS may hold NaNs
                const v8 v8v = __builtin_bit_cast(v8, vr);
#pragma unroll
                for (int e = 0; e < 8; ++e) acc[e] = fmaf(p, (float)v8v[e], acc[e]);
                l += p;
            }
            if (next) { if (LU && more) rows(vc_rs, nk0, njb, P_LU, P_AU, vv); else rows(vc_rs, nk0, njb, 0, P_AU, vv); }
        };
        int jb = 0;
        if constexpr (AHEAD) {
            if (k0 == 0 && nb > 0) { batch(std::true_type{}, 0); jb = 1; }
        }
        for (; jb < nb; ++jb) batch(std::false_type{}, jb);
        // the 8 key groups of a wave (lanes differing in bits 3..5), then the pair's four waves in order
        const float mw = max_rows(fmaxf(m, dpp<0x128>(m)));    // 0x128: rotated by eight within sixteen lanes
        const float f = __builtin_amdgcn_exp2f(m - (mw == -INFINITY ? 0.f : mw));
        l *= f;
        l = sum_rows(l + dpp<0x128>(l));
        // eight sums over eight groups: at each level a lane passes on the half of the values that it does not keep, and ends up with
        // elements e0 and e0 + 1 of its chunk
        float x4[4], x2[2];
#pragma unroll
        for (int e = 0; e < 4; ++e) x4[e] = add_halves32(acc[e] * f, acc[e + 4] * f);
#pragma unroll
        for (int e = 0; e < 2; ++e) { x2[e] = add_halves16(x4[e], x4[e + 2]); x2[e] += dpp<0x128>(x2[e]); }
        const int e0 = 4 * (c.lane >> 5) + 2 * ((c.lane >> 4) & 1);
        // With few pairs per member there is hardly ever a next one under way here, and the compiler should know: it would
        // wait at the start of the next stage, behind the stores of this one.
        if (MB == 1) __builtin_amdgcn_s_waitcnt(0x0F70);
        float *op = opart + par * (P_NW * 64);
        float2 *wp = wst + par * P_NW;
        par ^= 1;                                  // the other half may still be read by a slower wave
        if ((c.lane & 8) == 0) *reinterpret_cast<float2 *>(&op[c.wave * 64 + dc * 8 + e0]) = float2{x2[0], x2[1]};
        if (c.lane == 0) wp[c.wave] = float2{mw, l};
        __syncthreads();
        if (valid && stid < 64) {                  // one wave a pair, one element a lane
            const int w0 = 4 * sub;
            const float mm = fmaxf(fmaxf(wp[w0].x, wp[w0 + 1].x), fmaxf(wp[w0 + 2].x, wp[w0 + 3].x));
            float den = 0.f, sum = 0.f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float fw = __builtin_amdgcn_exp2f(wp[w0 + q].x - mm);
                den += wp[w0 + q].y * fw;
                sum += op[(w0 + q) * 64 + stid] * fw;
            }
            const float val = sum / den, other = dpp<0xB1>(val);       // the neighbour's element: two to a word
            typedef HT v2 __attribute__((ext_vector_type(2)));
            if ((stid & 1) == 0) {
                const int two = __builtin_bit_cast(int, v2{from_f32<HT>(val), from_f32<HT>(other)});
                const uint32_t eo = (uint32_t)frag_off(wsrow, h * 64 + stid, W / 32) * 2u;
                st4<ONE>(ws, out_off + eo, flagged(two));
                st4<ONE>(ws, empty_off + eo, -1);
            }
        }
    }
}

template <typename HT, int MB, int S, int CB, bool AHEAD, bool ONE>
__global__ __launch_bounds__(P_THREADS) void seq_persistent_kernel(SeqArgs a) {
    constexpr int W = 256 * S, RW_ROWS = 16 * MB, CBH = S <= 2 ? 2 : 4;
    constexpr int CBM = CB > CBH ? CB : CBH;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    __shared__ int sh[8];
    f32x4v *red = reinterpret_cast<f32x4v *>(lds_raw);                        // [8][CBM*MB][64]: LayerNorm-fused projections
    f32x4v *red2 = red + P_NW * CBM * MB * 64;                                // [8][MB][64]: residual projections
    float2 *stat = reinterpret_cast<float2 *>(red2 + P_NW * MB * 64);         // [8][MB*16]
    float2 *wst = stat + P_NW * MB * 16;                                      // [2][8]
    float *opart = reinterpret_cast<float *>(wst + 2 * P_NW);                 // [2][8][64]
    float *xs = opart + 2 * P_NW * 64;                                        // [16*MB][D]
    float *wemb = xs + RW_ROWS * a.D;                                         // [P_EB][D + 1][16]: w_in slice, then b_in
    float *pl = wemb + (size_t)P_EB * (a.D + 1) * 16;                         // [16*MB][2D]: this step's [mu | alpha] of the group's rows
    i32x4 *kv = reinterpret_cast<i32x4 *>(pl + (size_t)RW_ROWS * 2 * a.D);    // [2 P_LU][512]: cached rows for the next attention
    const uint32_t kv_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)kv;

    Ctx c;
    c.tid = threadIdx.x; c.lane = c.tid & 63; c.wave = c.tid >> 6; c.r = c.lane & 15; c.kg = c.lane >> 4;
    c.kv_stream = a.kv_stream != 0;
    c.status = a.sync + 9; c.spin_max = a.spin_max; c.bad = (LdsInt *)&sh[7];

    // ---- groups: the workgroups of xpg XCDs, found from the hardware's XCC id
    if (c.tid == 0) {
        const int xcc = __builtin_amdgcn_s_getreg(20 | (3 << 11)) & 7;  // HW_REG_XCC_ID, bits 3:0
        const int slot = atomicAdd(&a.sync[xcc], 1);
        // the arrival is a release and the poll an acquire (device scope, once per launch): a member that sees
        // every arrival also sees every member count, so all members of a group compute the same group size
        __hip_atomic_fetch_add(&a.sync[8], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        int it = 0, ok = 1;
        while (__hip_atomic_load(&a.sync[8], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < (int)gridDim.x) {
            if (++it > a.spin_max) { ok = 0; break; }
            __builtin_amdgcn_s_sleep(2);
        }
        int count[8];
        for (int g = 0; g < 8; ++g) count[g] = __hip_atomic_load(&a.sync[g], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
        const SeqGroup grp = seq_group_of(count, xcc, a.xpg, a.B, RW_ROWS);
        if (!ok) __hip_atomic_store(c.status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh[0] = ok; sh[1] = grp.before + slot; sh[2] = grp.members; sh[3] = grp.per; sh[4] = grp.index; sh[7] = 0;
    }
    __syncthreads();
    if (!sh[0]) return;
    c.slot = sh[1]; c.n = sh[2];
    const int per = sh[3], gidx = sh[4];           // samples per group
    if (per > RW_ROWS) {                           // too few XCDs for the batch
        if (c.tid == 0) __hip_atomic_store(c.status, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    c.row0 = gidx * per;
    c.nrows = a.B - c.row0 < per ? a.B - c.row0 : per;
    c.rb0 = gidx * MB;
    c.cw = W / 4 <= c.n ? 4 : (W / 8 <= c.n ? 8 : 16);
    if (c.nrows <= 0) return;                      // groups are independent: an idle one just leaves
    // a member without a share of any stage leaves as well: nobody reads anything of it
    // (the MLP input has the most column blocks, W / 4; a unit of the residual projections has at least four columns)
    if (c.slot >= W / 4 && c.slot >= c.nrows * (W / 64)) return;

    const int T = a.T, D = a.D;
    constexpr uint32_t UW = 8u * RW_ROWS * W;      // elements of one slot of a buffer of width W
    const rsrc_t ws = make_rsrc(a.ws, UW * kSeqWsBytesPerElem);
    auto off_h = [&](int s) { return (uint32_t)(s & 3) * (4u * UW); };                  // stream: embedding, MLP output
    auto off_a = [&](int s) { return (16u + (uint32_t)s * 4u) * UW; };                  // stream: attention output
    auto off_q = [&](int s) { return (28u + (uint32_t)s * 6u) * UW; };
    auto off_o = [&](int s) { return (46u + (uint32_t)s * 2u) * UW; };
    auto off_f = [&](int s) { return (52u + (uint32_t)s * 8u) * UW; };
    const int cw = c.cw, nu = W / cw;
    // this member's slices of the embedding matrix and bias stay in LDS for the whole block
    for (int bi = 0, u = c.slot; bi < P_EB && u < nu; ++bi, u += c.n)
        for (int e = c.tid; e < (D + 1) * cw; e += P_THREADS) {
            const int d = e / cw, cl = e - d * cw;
            wemb[bi * (D + 1) * 16 + e] = d < D ? a.w_in[(size_t)d * W + u * cw + cl] : a.b_in[u * cw + cl];
        }
    // latent values of position 0 (each thread keeps the ones it will turn into x), position embedding likewise
    constexpr int ZPT = (RW_ROWS * 64 + P_THREADS - 1) / P_THREADS;   // token sizes up to 64
    float zreg[ZPT];
#pragma unroll
    for (int q = 0; q < ZPT; ++q) {
        const int e = c.tid + q * P_THREADS;
        zreg[q] = 0.f;
        if (e < RW_ROWS * D) {
            const int row = e / D, d = e - row * D;
            if (row < c.nrows) zreg[q] = a.z[((size_t)(c.row0 + row) * T + (a.reversed ? T - 1 : 0)) * D + d];
        }
    }
    const int er = c.tid / cw, ec = c.tid - er * cw;     // embedding: row and column of a unit (512 threads: 32 x 16 at most)
    float pos0 = c.slot < nu ? a.pos[c.slot * cw + ec] : 0.f;
    __syncthreads();

    int s3 = 0, hq = 0, par = 0;
    for (int l = 0; l < T; ++l) {
        // ---- x_l of the group's samples (eq. 5; x_0 = z_0), kept in LDS for the embedding; the latent
        // values were requested one step ahead
        const int tok = a.reversed ? T - 1 - l : l;
        const int tok_next = a.reversed ? T - 2 - l : l + 1;
#pragma unroll
        for (int q = 0; q < ZPT; ++q) {
            const int e = c.tid + q * P_THREADS;
            if (e < RW_ROWS * D) {
                const int row = e / D, d = e - row * D;
                float xn = 0.f;
                if (row < c.nrows) {
                    const size_t idx = ((size_t)(c.row0 + row) * T + tok) * D + d;
                    xn = zreg[q];
                    if (l > 0) xn = fmaf(xn, expf(pl[row * 2 * D + D + d]), pl[row * 2 * D + d]);
                    if (c.slot == 0) a.x[idx] = xn;
                    if (l + 1 < T) zreg[q] = a.z[((size_t)(c.row0 + row) * T + tok_next) * D + d];
                }
                xs[e] = xn;
            }
        }
        if (l == T - 1) break;
        __syncthreads();
        // ---- embedding of this member's units: stream = x_l * w_in + b_in + pos[l]
        {
            int bi = 0;
            for (int u = c.slot; u < nu; u += c.n, ++bi) {
                const int col = u * cw + ec;
                if (er < c.nrows) {
                    float acc = bi == 0 ? pos0 : a.pos[(size_t)l * W + col];
                    if (bi < P_EB) {
                        const float *we = wemb + bi * (D + 1) * 16;
                        acc += we[D * cw + ec];
                        for (int d = 0; d < D; ++d) acc = fmaf(xs[er * D + d], we[d * cw + ec], acc);
                    } else {
                        acc += a.b_in[col];
                        for (int d = 0; d < D; ++d) acc = fmaf(xs[er * D + d], a.w_in[(size_t)d * W + col], acc);
                    }
                    const uint32_t eo = (uint32_t)frag_off(c.rb0 * 16 + er, col, W / 32) * 4u;
                    st4<ONE>(ws, off_h(hq) + eo, flagged(acc));
                    st4<ONE>(ws, off_h(hq + 2) + eo, -1);            // slot of use hq - 2
                    if (bi == 0 && l + 1 < T) pos0 = a.pos[(size_t)(l + 1) * W + col];
                }
            }
        }
        for (int ly = 0; ly < a.n_layers; ++ly) {
            const SeqLayer &lw = a.layers[ly];
            HT *kc = reinterpret_cast<HT *>(a.kcache) + (size_t)ly * a.kv_layer_stride;
            HT *vc = reinterpret_cast<HT *>(a.vcache) + (size_t)ly * a.kv_layer_stride;
            const rsrc_t kc_rs = make_rsrc(kc, (uint32_t)(a.kv_layer_stride * 2u));
            const rsrc_t vc_rs = make_rsrc(vc, (uint32_t)(a.kv_layer_stride * 2u));
            const int e3 = s3 == 0 ? 2 : s3 - 1;                // slot of the use before this one
            // cached rows for the next attention: part 3 (behind the QKV projection) for this layer's, parts 0 to 2 for that of the next
            // layer or of the next step's first
            auto ahead = [&](int part) {
                return [&, part]() { (void)part;
                    if constexpr (AHEAD) {
                        const int next = part == 3 ? ly : ly + 1;
                        const bool wrap = next == a.n_layers;
                        const size_t off = wrap ? 0 : (size_t)next * a.kv_layer_stride;
                        kv_ahead<S>(c, part, reinterpret_cast<const HT *>(a.kcache) + off, reinterpret_cast<const HT *>(a.vcache) + off,
                                    wrap ? l + 1 : l, T, kv_lds);
                    }
                };
            };
            ln_gemm_stage<HT, MB, S, CB, EPI_BIAS, false, ONE>(c, ws, off_h(hq), lw.ln1_g, lw.ln1_b, (const HT *)lw.f_qkv, lw.b_qkv,
                                                               off_q(s3), off_q(e3), nullptr, 3 * W, red, stat, ahead(3));
            attention_stage<HT, MB, S, AHEAD, ONE>(c, ws, off_q(s3), kc, vc, kc_rs, vc_rs, off_o(s3), off_o(e3), l, T, opart, wst, par, kv);
            gemm_resid_stage<HT, MB, S, 1, ONE>(c, ws, off_o(s3), (const HT *)lw.f_o, lw.b_o, off_h(hq), off_a(s3), off_a(e3), red2, ahead(0));
            ln_gemm_stage<HT, MB, S, CB, EPI_BIAS_GELU, false, ONE>(c, ws, off_a(s3), lw.ln2_g, lw.ln2_b, (const HT *)lw.f_fc1, lw.b_fc1,
                                                                    off_f(s3), off_f(e3), nullptr, 4 * W, red, stat, ahead(1));
            gemm_resid_stage<HT, MB, S, 4, ONE>(c, ws, off_f(s3), (const HT *)lw.f_fc2, lw.b_fc2, off_a(s3), off_h(hq + 1), off_h(hq + 3), red2, ahead(2));
            ++hq;
            s3 = s3 == 2 ? 0 : s3 + 1;
        }
        // ---- head: every member computes all of [mu | alpha] for the group's rows (a few column blocks)
        // into its own LDS, so that x_l and the next embedding follow without another exchange
        ln_gemm_stage<HT, MB, S, CBH, EPI_BIAS, true, ONE>(c, ws, off_h(hq), a.lnf_g, a.lnf_b, (const HT *)a.f_head, a.b_head, 0, 0,
                                                           pl, 2 * D, red, stat, []() {});
        ++hq;
        __syncthreads();
        if (*c.bad) return;
    }
}

// Every buffer empty, the synchronisation words zero (a kernel: memory operations of the runtime stay out of the path).
__global__ __launch_bounds__(256) void seq_reset_kernel(uint4 *ws, size_t n16, int *sync) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256)
        ws[i] = uint4{kEmpty, kEmpty, kEmpty, kEmpty};
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < kSeqSyncWords; i += 256) sync[i] = 0;
}

}  // namespace

static size_t seq_lds_bytes(int MB, int D, bool ahead) {
    const size_t need = (ahead ? P_AHEAD_BYTES : 0) + (size_t)P_NW * 4 * MB * 64 * 16 + (size_t)P_NW * MB * 64 * 16 + (size_t)P_NW * MB * 16 * 8 + 2 * P_NW * 8 +
                        (size_t)2 * P_NW * 64 * 4 + (size_t)16 * MB * D * 4 + (size_t)P_EB * (D + 1) * 16 * 4 + (size_t)16 * MB * 2 * D * 4;
    const size_t one_per_cu = 84 * 1024;  // more than half of a CU's LDS: exactly one workgroup per CU
    return ((need < one_per_cu ? one_per_cu : need) + 255) & ~(size_t)255;
}

size_t seq_persistent_lds_bytes(int MB, int D) { return seq_lds_bytes(MB, D, MB == 1); }

template <typename HT>
static const void *pick_kernel(int MB, int S, int CB, bool ahead, bool one) {
#define SJD_PK(MBv, Sv, CBv, AHv, ONEv) if (MB == MBv && S == Sv && CB == CBv && ahead == AHv && one == ONEv) return reinterpret_cast<const void *>(&seq_persistent_kernel<HT, MBv, Sv, CBv, AHv, ONEv>);
    // one XCD per group: a member has two column blocks of the MLP input or more; width 256 knows no other groups
#define SJD_ONE(Sv) SJD_PK(1, Sv, 4, false, true) SJD_PK(2, Sv, 4, false, true)
#define SJD_ANY(Sv) SJD_PK(1, Sv, 1, false, false) SJD_PK(1, Sv, 2, false, false) SJD_PK(1, Sv, 4, false, false)
    SJD_PK(1, 1, 2, false, true)
    SJD_ONE(1) SJD_ONE(2) SJD_ONE(3) SJD_ONE(4) SJD_ANY(2) SJD_ANY(3) SJD_ANY(4)
    // cached rows ahead: a member has a second pair, so its group is no larger than that leaves it two column blocks (width 512: four)
    SJD_PK(1, 2, 4, true, true) SJD_PK(1, 3, 4, true, true) SJD_PK(1, 4, 4, true, true)
    SJD_PK(1, 2, 4, true, false) SJD_PK(1, 3, 2, true, false) SJD_PK(1, 3, 4, true, false) SJD_PK(1, 4, 2, true, false) SJD_PK(1, 4, 4, true, false)
#undef SJD_ANY
#undef SJD_ONE
#undef SJD_PK
    return nullptr;
}

hipError_t launch_seq_persistent(bool is_bf16, const SeqArgs &args, int MB, int S, int grid, bool cooperative,
                                 hipStream_t s) {
    // column blocks of a LayerNorm-fused projection per round: as many as a member of a group has of the widest one
    const int members = grid / 8 * args.xpg, blocks = 64 * S;
    const int per = members > 0 ? (blocks + members - 1) / members : blocks;
    const bool one = args.xpg == 1;
    const int CB = MB == 2 || per > 2 ? 4 : one && per < 2 ? 2 : per;
    const bool ahead = args.kv_ahead != 0;
    const void *kern = is_bf16 ? pick_kernel<bf16>(MB, S, CB, ahead, one) : pick_kernel<f16>(MB, S, CB, ahead, one);
    if (!kern) return hipErrorInvalidValue;
    const size_t lds = seq_lds_bytes(MB, args.D, ahead);
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(seq_reset_kernel, dim3(512), dim3(256), 0, s, (uint4 *)args.ws,
                       seq_persistent_ws_bytes(MB, 256 * S) / 16, args.sync);
    SeqArgs a = args;
    void *params[] = {&a};
    if (cooperative) return hipLaunchCooperativeKernel(kern, dim3(grid), dim3(P_THREADS), params, (unsigned)lds, s);
    // plain launch: co-residency of the workgroups is then not guaranteed by the runtime; it holds when
    // the device is otherwise idle (one workgroup per CU), and every wait in the kernel is bounded
    return hipLaunchKernel(kern, dim3(grid), dim3(P_THREADS), params, lds, s);
}

}  // namespace sjd

// MLP-input projection with GELU, C[M,N] (16-bit) = gelu(A[M,K] * W + bias), for launches that fill the chip: two persistent workgroups per CU.
//
// What bounds this projection: the matrix instructions, which power holds at about 1.3 PFLOP/s on random operands whatever feeds them (212 us of
// 32768 x 4096 x 1024; four waves of 128 x 128, operands from L2 instead of LDS, one workgroup or two all give the same), and GELU: fifteen
// issue slots a value, 54 us of vector ALU in that launch, which the persistent kernel of gemm_p8.hip cannot run beside matrix instructions,
// for its one workgroup per CU has all of its accumulators in the epilogue at once.  Here a CU holds two independent workgroups, a 128 x
// 256 tile and 80 KB of LDS each, so that one works on its epilogue while the other multiplies.  They start in step; the second half of a tile's k
// and its epilogue run at a higher wave priority, so that of two the one that is ahead finishes first and they fall out of step within a tile or
// two.  (Priority lowered before the epilogue: 13659 x 4096 x 1024 114.4 -> 112.7 us, 18139 x 3072 x 768 92.0 -> 90.8, 26587 x 3072 x 768 129.1 -> 131.3, 27355 x
// 2048 x 512 70.3 -> 71.3.)
//   * four waves per workgroup, one per SIMD, 128 x 64 of the tile each (128 accumulator registers);
//   * A through LDS: k-tiles of 64 (whole cache lines) in a ring of four 16 KB units filled by LDS-direct loads three k-tiles ahead, one
//     barrier per k-tile; swizzled as in gemm_p8.hip;
//   * weights in the fragment order of the 32x32x16 instruction (launch_weights_to_frag32), from L2 straight into registers, eight k-steps
//     ahead: a smaller tile needs more operand bytes per product, and LDS could not deliver both;
//   * both request streams run on into the workgroup's next tile; the epilogue parks accumulators in 16 KB of LDS of its own.
// k is walked in index order with the same instruction: results are bit-identical to the other 16-bit kernels.
// Measured alone, us, gemm_p8.hip -> this: 32768 x 4096 x 1024 276 -> 257, 16384 x 4096 x 1024 143 -> 133, 65536 x 3072 x 768 340 -> 301, 8192 x 3072 x 768
// 55 -> 45, 32768 x 2048 x 512 91 -> 83; inside the passes of the largest flows 1.5 to 2 %.  The other epilogues gain nothing or lose (float32 residual at k
// = 4096: 246 -> 257).
#include "common.h"
#include "gemm_rules.h"
#include <atomic>
#include <type_traits>

namespace sjd {

namespace {

constexpr int U_BM = kDuoRows, U_BN = kDuoCols;
constexpr int U_CB = 4;                       // column tiles per column block of the tile order
constexpr int U_UNITS = 4, U_UNIT = 16 * 1024;  // units of the LDS ring: A of one k-tile, 128 rows x 128 B
constexpr int U_PARK = 16 * 1024;
constexpr int U_LDS = U_UNITS * U_UNIT + U_PARK;   // 80 KB: two workgroups per CU
constexpr int U_PD = 8;                       // weight fragments on their way, in k-steps
constexpr int kOutside = 0x7FFFFFF0;          // a lane offset past any buffer range this kernel declares

typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef int i32x2 __attribute__((ext_vector_type(2)));

template <typename HT>
__global__ __launch_bounds__(256, 2) void gemm_h16_duo_kernel(const HT *__restrict__ A, const HT *__restrict__ Wf,
                                                              const float *__restrict__ bias, HT *C, int M, int N,
                                                              int K, int tiles_m, int tiles_n, int col_block) {
    typedef typename Half16<HT>::v8 v8;
    typedef typename Half16<HT>::v4 v4;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    // Tile order of gemm_p8.hip: an XCD (workgroup id mod 8) owns a range of row panels and walks it in blocks of four column tiles.
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, n_slots = gridDim.x >> 3;
    const int rp0 = (int)((long long)xcd * tiles_m / 8), nrp = (int)((long long)(xcd + 1) * tiles_m / 8) - rp0;
    const int n_mine = nrp * tiles_n;
    auto tile_of = [&](int li) {
        if (li >= n_mine) return -1;
        const int cb = li / (nrp * col_block);
        const int left = tiles_n - cb * col_block, cbw = left < col_block ? left : col_block;
        const int lo = li - cb * nrp * col_block;
        const int r = lo / cbw;
        return (rp0 + r) * tiles_n + cb * col_block + (lo - r * cbw);
    };
    int li = slot;
    int tile = tile_of(li);
    if (tile < 0) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, g = lane >> 5;
    const int KT = K / 64, KS16 = K / 16;
    // A: per k-tile a wave brings the 8-row blocks 4 wave + q, lane 8 r + c the chunk that belongs in slot c of row r; chunk c of row r lies in
    // slot c ^ swz(r), swz = bits 1, 2 and 4 of r.  Addresses: a uniform base plus 32-bit lane offsets.
    const int lr = lane >> 3;
    const int lc0 = (lane & 7) ^ ((lr >> 1) & 3);
    const uint32_t row_bytes = (uint32_t)K * 2u;
    struct Src { uint32_t off[4]; const char *base; };
    auto make_src = [&](int t) {
        Src s;
        const int tm = t / tiles_n;
        const int last = M - 1 - tm * U_BM;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int row = (wave * 4 + i) * 8 + lr;
            row = row < last ? row : last;                       // rows past the end: re-read the last row, never stored
            s.off[i] = (uint32_t)row * row_bytes + (uint32_t)((lc0 ^ (((i >> 1) & 1) << 2)) * 16);
        }
        s.base = reinterpret_cast<const char *>(A + (size_t)tm * U_BM * K);
        return s;
    };
    auto dma = [&](const char *base, uint32_t off, uint32_t lds_addr) {    // nothing else in this kernel reads M0
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :: "s"(lds_addr), "v"(off), "s"(base) : "memory");
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)lds;
    auto issue_a = [&](const Src &s, int kt, int unit, int q) {
        dma(s.base + (size_t)kt * 128, s.off[q], lds0 + (uint32_t)(unit * U_UNIT + (wave * 4 + q) * 1024));
    };
    const int swz = ((l32 >> 1) & 3) | (((l32 >> 4) & 1) << 2);
    int fk[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) fk[ks] = l32 * 128 + (((2 * ks + g) ^ swz) << 4);
    v8 fa[4], fb[U_PD][2];
    auto read_a = [&](int unit, int ks, int i) {
        fa[i] = *reinterpret_cast<const v8 *>(lds + unit * U_UNIT + 32 * i * 128 + fk[ks]);
    };
    const rsrc_t b_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<HT *>(Wf), 0, N * K * 2, 0x00020000);
    const int lane16 = lane * 16;
    auto b_tile = [&](int t) { const int tn = t - t / tiles_n * tiles_n; return (tn * 8 + wave * 2) * KS16 * 1024; };
    auto load_b = [&](int base, int ks, int j) {
        fb[ks % U_PD][j] = __builtin_bit_cast(v8, __builtin_amdgcn_raw_buffer_load_b128(b_rs, lane16, base + (j * KS16 + ks) * 1024, 0));
    };
    f32x16 acc[4][2];
    // Two k-tiles from unit ra on: 64 matrix instructions of this wave, each a slot with its LDS reads and loads pinned.  A of the k-tiles three
    // ahead (s0 / kt0, s1 / kt1) goes to the unit that the k-tile before left, a weight fragment is requested again for the next pair (bb)
    // as soon as its last use has been issued.  Behind the second slot of a k-tile's last k-step all of its fragments are in registers: wait for
    // this wave's part of the next k-tile (requested two k-tiles ago; 28 loads are younger, so all but the twelve
    // youngest is enough), then the barrier.
    auto kpair = [&](auto first, const Src &s0, int kt0, const Src &s1, int kt1, int bb, int ra) {
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
            const int unit = (ra + t2) & 3, unit_n = (ra + t2 + 1) & 3, unit_l = (ra + t2 + 3) & 3;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const int st = 4 * t2 + ks;
                const bool last = ks == 3;
                const int ua = last ? unit_n : unit, rk = last ? 0 : ks + 1;
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    const int i = m >> 1, j = m & 1;
                    if (decltype(first)::value && st == 0) acc[i][j] = Half16<HT>::mfma(fa[i], fb[0][j], f32x16{});
                    else acc[i][j] = Half16<HT>::mfma(fa[i], fb[st][j], acc[i][j]);
                    __builtin_amdgcn_sched_barrier(0);
                    if (last && m == 1) {
                        __builtin_amdgcn_s_waitcnt(0x0074 | 8);   // vmcnt(12) lgkmcnt(0)
                        __builtin_amdgcn_s_barrier();
                    }
                    if (j == 1) read_a(ua, rk, i);
                    if (ks < 2 && (m == 2 || m == 6)) issue_a(t2 ? s1 : s0, t2 ? kt1 : kt0, unit_l, 2 * ks + (m >> 2));
                    if (m >= 6) load_b(bb, st, j);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    };
    Src cur = make_src(tile);
    int bcur = b_tile(tile);
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int q = 0; q < 4; ++q) issue_a(cur, t, t, q);
#pragma unroll
    for (int sl = 0; sl < U_PD; ++sl) { load_b(bcur, sl, 0); load_b(bcur, sl, 1); }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i) read_a(0, 0, i);
    int ra = 0;
    const int rl = lane >> 4, cl = (lane & 15) * 4;
    float *ep = reinterpret_cast<float *>(lds + U_UNITS * U_UNIT) + wave * 1024;
    while (true) {
        const int tm = tile / tiles_n, tn = tile - tm * tiles_n;
        li += n_slots;
        const int tile_next = tile_of(li);
        // no next tile: request this tile's first k-tiles again (in bounds, never used)
        const Src nxt = make_src(tile_next >= 0 ? tile_next : tile);
        const int bnxt = b_tile(tile_next >= 0 ? tile_next : tile);
        auto pair_at = [&](auto first, int kt) {
            const bool w0 = kt + 3 >= KT, w1 = kt + 4 >= KT;
            Src s0, s1;
#pragma unroll
            for (int i = 0; i < 4; ++i) { s0.off[i] = w0 ? nxt.off[i] : cur.off[i]; s1.off[i] = w1 ? nxt.off[i] : cur.off[i]; }
            s0.base = w0 ? nxt.base : cur.base; s1.base = w1 ? nxt.base : cur.base;
            const int bb = kt + 2 >= KT ? bnxt : bcur + (kt + 2) * 4096;
            kpair(first, s0, w0 ? kt + 3 - KT : kt + 3, s1, w1 ? kt + 4 - KT : kt + 4, bb, ra);
            ra = (ra + 2) & 3;
        };
        __builtin_amdgcn_s_setprio(0);
        pair_at(std::true_type{}, 0);
        for (int kt = 2; kt < KT; kt += 2) {
            if (kt >= KT / 2) __builtin_amdgcn_s_setprio(1);
            pair_at(std::false_type{}, kt);
        }
        // ---- epilogue, as in gemm_p8.hip: sixteen rows x 64 columns at a time through the wave's parking slice, back row-wise, four columns a
        // lane; rows past M are dropped by the buffer's bounds.
        {
            const int row0 = tm * U_BM, col0 = tn * U_BN + wave * 64;
            int rows_left = M - row0;
            rows_left = rows_left > 128 ? 128 : rows_left;
            HT *cbase = C + (size_t)row0 * N + col0;
            const int n_bytes = ((rows_left - 1) * N + 64) * (int)sizeof(HT);
            const rsrc_t c_rs = __builtin_amdgcn_make_buffer_rsrc(cbase, 0, n_bytes, 0x00020000);
            int lane_off = (rl * N + cl) * (int)sizeof(HT);
            asm volatile("" : "+v"(lane_off));
            const int row_step = N * (int)sizeof(HT);
            const f32x4 bv4 = *reinterpret_cast<const f32x4 *>(bias + col0 + cl);
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                const int i = n >> 1, hh = n & 1;
                f32x4 val[4];
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int vv = 0; vv < 8; ++vv)
                        ep[(8 * (vv >> 2) + 4 * g + (vv & 3)) * 64 + 32 * (j ^ g) + l32] = acc[i][j][8 * hh + vv];
                asm volatile("" ::: "memory");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    val[q] = *reinterpret_cast<const f32x4 *>(&ep[(4 * q + rl) * 64 + (cl ^ (32 * (q & 1)))]);
                asm volatile("" ::: "memory");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int r0 = 32 * i + 16 * hh + 4 * q;
                    const int s_off = r0 * row_step;
                    const int v_off = r0 + rl < rows_left ? lane_off : kOutside;
                    f32x4 o = val[q] + bv4;
                    v4 o4;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o4[e] = from_f32<HT>(gelu_erf_h16(o[e]));
                    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2, o4), c_rs, v_off, s_off, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (tile_next < 0) break;
        bcur = bnxt;
        tile = tile_next;
        cur = nxt;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);       // the loads of the unused last requests have landed before the LDS goes away
}

}  // namespace

template <typename HT>
void launch_gemm_duo_gelu(const HT *A, const HT *Wf, const float *bias, HT *C, int M, int N, int K, hipStream_t s) {
    const int tiles_m = (M + U_BM - 1) / U_BM, tiles_n = N / U_BN;
    const int per_xcd = ((tiles_m + 7) / 8) * tiles_n;      // tiles of the XCD with the most row panels
    const int slots = per_xcd < 64 ? per_xcd : 64;          // two workgroups on each of 32 CUs
    auto kern = gemm_h16_duo_kernel<HT>;
    static std::atomic<bool> attr_set{false};               // callers may come from several host threads
    if (!attr_set.load(std::memory_order_acquire)) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, U_LDS);
        attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3(8 * slots), dim3(256), U_LDS, s, A, Wf, bias, C, M, N, K, tiles_m, tiles_n, U_CB);
}
template void launch_gemm_duo_gelu<bf16>(const bf16 *, const bf16 *, const float *, bf16 *, int, int, int, hipStream_t);
template void launch_gemm_duo_gelu<f16>(const f16 *, const f16 *, const float *, f16 *, int, int, int, hipStream_t);

}  // namespace sjd

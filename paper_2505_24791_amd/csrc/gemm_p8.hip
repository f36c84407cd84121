// Persistent 16-bit MFMA projection, eight waves per workgroup: C[M,N] = epi(A[M,K] * Bt[N,K]^T + bias).
//
// The tile kernels of gemm_h16.hip run one tile per workgroup: every tile pays its first loads and the
// drain of its epilogue's stores in full, because the next workgroup cannot start on the CU before this
// one has gone (128 KB of LDS each).  Here one workgroup per CU stays resident and walks over its tiles:
//   * 256 x 256 output tile; k-tiles of 64, so that a row's piece of a k-tile is a whole 128-byte cache line: with
//     k-tiles of 32 every line was asked of L2 twice, half a line at a time (34 M requests per launch at M = 32768,
//     N = 1024, K = 4096 against 17 M now, for the same bytes), and L2 requests were what the kernel waited for;
//   * one operand of one k-tile is a unit of 32 KB; five units form a ring in LDS, filled by LDS-direct loads
//     (no staging registers): while k-tile t is multiplied (two units), k-tile t + 1 and the A operand of
//     t + 2 land, so a load has one to two k-tiles to arrive and the requests are spread over the k-tile;
//   * eight waves, two per SIMD, each owning 128 x 64 of the tile (128 accumulator registers);
//   * the request stream runs on across tiles: the first k-tiles of the NEXT tile are requested during
//     the last ones of this tile and the first has landed before the epilogue starts, so a tile begins with
//     operands already in LDS;
//   * the epilogue parks accumulators in the one unit that is free at that time, so the others keep
//     filling meanwhile, and its stores drain while the next tile multiplies.
// k is walked in index order with the 32x32x16 instruction, an output row depends on its own row of A
// only: results are bit-identical to the tile kernels and independent of the batch.
// Covers K % 64 == 0, K >= 128 and N % 256 == 0 (every projection of the workloads but the head).
// Measured (us per launch, k-tiles of 32 in four stages -> this; IEEE half, bias / GELU / float32 residual epilogue):
//   32768 x 3072 x 1024 bias 197 -> 178, 32768 x 4096 x 1024 GELU 300 -> 278, 32768 x 1024 x 1024 residual 101 -> 85,
//   32768 x 1024 x 4096 residual 281 -> 246, 65536 x 768 x 3072 residual 337 -> 297.
// What bounds it: power, then the epilogues.  Without its epilogue the kernel runs at 1.25 to 1.30 PFLOP/s on random operands at all of
// these shapes (1.7 on a zero left operand), and so do variants with the weights from L2 instead of LDS, with two workgroups of four waves, and with the waits
// taken out; four waves of 128 x 128 (a third fewer LDS reads) take as long with more idle cycles at a higher clock.  On top come the epilogues: bias 16 us
// of the first shape, a float32 residual 30 of the third and fourth (all CUs read and write 256 KB each at once; starting them staggered, and residual loads
// one to three groups ahead, gained nothing), GELU 63 of the second, 54 of them vector ALU: launches with GELU that fill the chip go to gemm_duo.hip, which
// runs it beside the matrix instructions.
#include "common.h"
#include <atomic>

namespace sjd {

namespace {

constexpr int Q_BM = 256, Q_BN = 256;
constexpr int Q_CB = 4;                     // column tiles per column block of the tile order
constexpr int D_BK = 64, D_KSUB = D_BK / 16;  // k-tile, k-steps per k-tile
constexpr int D_UNITS = 5;                  // units of the LDS ring
constexpr int D_OPB = 32 * 1024;            // bytes of a unit: one operand of one k-tile, 256 rows x 128 B
constexpr int D_LDS = D_UNITS * D_OPB;      // 160 KB
constexpr int kOutside = 0x7FFFFFF0;        // a lane offset past any buffer range this kernel declares

typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

#define SJD_Q_LPTR(p) ((__attribute__((address_space(3))) void *)(p))

template <typename HT, typename OutT, int EPI>
__global__ __launch_bounds__(512) void gemm_h16_p8_kernel(const HT *__restrict__ A, const HT *__restrict__ Bt,
                                                             const float *__restrict__ bias, OutT *C, int M, int N,
                                                             int K, int tiles_m, int tiles_n, int col_block) {
    typedef typename Half16<HT>::v8 v8;
    typedef typename Half16<HT>::v4 v4;
    constexpr bool OUT_F32 = sizeof(OutT) == 4;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    // Workgroup ids congruent mod 8 share an XCD (and its L2).  Each XCD owns a contiguous range of row panels
    // and walks it column block by column block (Q_CB column tiles wide), row by row inside a block; its
    // workgroups take the tiles of that order round-robin.  So at any time the 32 workgroups of an XCD work on
    // about eight row panels against the same few column tiles of the weight, and the next round keeps those
    // column tiles: the weight rows of a column block (2 MB at k = 1024) stay in the 4 MB L2 while the row
    // panels stream past them, instead of the whole weight being fetched again for every pair of row panels
    // (measured on the MLP input projection, M = 32768, N = 4096, K = 1024: 637 MB per launch went through the
    // L2-miss counters in plain row-major tile order, for 75 MB of operands; blocks of 4 column tiles are
    // 5-10 % faster than row-major order on the q/k/v and MLP input shapes, blocks of 2 are slower, 6 the same).
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
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: LDS bases stay in scalar registers
    const int l32 = lane & 31, g = lane >> 5;
    const int wm = wave >> 2, wn = wave & 3;                     // this wave's 128 x 64 part of the tile
    const int KT = K / D_BK;

    // Loads.  A unit holds 256 rows of 128 bytes (eight 16-byte chunks).  Per unit a wave brings the 8-row blocks
    // 4 wave + q (q = 0..3), 1 KB each: lane 8 r + c delivers the chunk that belongs in slot c of row r.  Row r of
    // a 32-row fragment group keeps chunk c in slot c ^ swz(r), swz(r) = bits 1, 2 and 4 of r: a 16-byte LDS read of
    // a wave is served in four passes of 16 lanes (rows {0-7, 16-23} or {8-15, 24-31} of the group, one chunk) over
    // 64 banks; with rows 128 bytes apart the bank group of a read is 8 (r mod 2) + slot, which this makes distinct
    // over the sixteen rows of a pass.
    // Addresses are a wave-uniform 64-bit base (the tile's first row, advanced by the k-tile) plus a
    // per-lane 32-bit byte offset inside the tile: few registers, and no 32-bit overflow however large M is.
    const int lr = lane >> 3;                                    // row within the 8-row block
    const int lc0 = (lane & 7) ^ ((lr >> 1) & 3);                // chunk fetched for blocks with bit 4 of the row clear
    const uint32_t row_bytes = (uint32_t)K * 2u;
    struct Src { uint32_t a_off[4]; const char *a_base, *b_base; };
    auto make_src = [&](int t) {
        Src s;
        const int tm = t / tiles_n, tn = t - tm * tiles_n;
        const int last = M - 1 - tm * Q_BM;                      // last valid row of this tile (tile-relative, >= 0)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int row = (wave * 4 + i) * 8 + lr;
            row = row < last ? row : last;                       // rows past the end: re-read the last row, never stored
            s.a_off[i] = (uint32_t)row * row_bytes + (uint32_t)((lc0 ^ (((i >> 1) & 1) << 2)) * 16);
        }
        s.a_base = reinterpret_cast<const char *>(A + (size_t)tm * Q_BM * K);
        s.b_base = reinterpret_cast<const char *>(Bt + (size_t)tn * Q_BN * K);   // Bt rows are padded to the tile
        return s;
    };
    uint32_t b_off[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        b_off[i] = (uint32_t)((wave * 4 + i) * 8 + lr) * row_bytes + (uint32_t)((lc0 ^ (((i >> 1) & 1) << 2)) * 16);
    // An LDS-direct load: 64 lanes x 16 bytes from (wave-uniform base) + (per-lane 32-bit offset) to 1 KB of LDS
    // at the wave-uniform byte address lds_addr (through M0).  Written out so that the address stays split
    // into a scalar base and a 32-bit lane offset (two registers per lane per load otherwise).  M0 is set
    // inside the statement and nothing else in this kernel reads it (no other LDS-direct access, no
    // indexed register moves), so nothing of the compiler's is lost.
    auto dma = [&](const char *base, uint32_t off, uint32_t lds_addr) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                     :: "s"(lds_addr), "v"(off), "s"(base) : "memory");
    };
    const uint32_t lds0 = (uint32_t)(uintptr_t)SJD_Q_LPTR(lds);
    auto issue_a = [&](const Src &s, int kt, int unit, int q) {
        dma(s.a_base + (size_t)kt * (D_BK * 2), s.a_off[q], lds0 + (uint32_t)(unit * D_OPB + (wave * 4 + q) * 1024));
    };
    auto issue_b = [&](const Src &s, int kt, int unit, int q) {
        dma(s.b_base + (size_t)kt * (D_BK * 2), b_off[q], lds0 + (uint32_t)(unit * D_OPB + (wave * 4 + q) * 1024));
    };
    // Fragments: row l32 of a 32-row group, chunk 2 ks + g, found in slot (2 ks + g) ^ swz(l32); rows are 128 B
    // apart.  A fragments are refreshed in place right after their last use in a k-step, B fragments
    // (used by all four row groups) alternate between two sets.
    const int swz = ((l32 >> 1) & 3) | (((l32 >> 4) & 1) << 2);
    int fk[D_KSUB];
#pragma unroll
    for (int ks = 0; ks < D_KSUB; ++ks) fk[ks] = l32 * 128 + (((2 * ks + g) ^ swz) << 4);
    const int a_lds = wm * (128 * 128), b_lds = wn * (64 * 128);
    v8 fa[4], fb[2][2];
    auto read_a = [&](int unit, int ks, int i) {
        fa[i] = *reinterpret_cast<const v8 *>(lds + (unit * D_OPB + a_lds) + 32 * i * 128 + fk[ks]);
    };
    auto read_b = [&](int unit, int ks, int buf, int j) {
        fb[buf][j] = *reinterpret_cast<const v8 *>(lds + (unit * D_OPB + b_lds) + 32 * j * 128 + fk[ks]);
    };

    f32x16 acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // One k-tile t: 32 matrix instructions of this wave, each a slot with its LDS reads and loads pinned.  Its operands
    // are units ra and ra + 1 (mod 5), those of t + 1 are ra + 2 and ra + 3.  The A operand of t + 2 (`next` / `next_kt`)
    // goes to unit ra + 4 during the first two k-steps.  After the second slot of the last k-step, when all of this
    // k-tile's fragments are in registers: wait until this wave's loads of k-tile t + 1 have landed (the four
    // younger ones may stay in flight: loads complete in order), then the barrier; the rest of the k-step reads the
    // next k-tile's first fragments and requests the B operand of t + 2 into unit ra.
    auto up = [](int u, int d) { u += d; return u >= D_UNITS ? u - D_UNITS : u; };
    auto ktile = [&](int ra, const Src &next, int next_kt) {
        const int rb = up(ra, 1), ra1 = up(ra, 2), rb1 = up(ra, 3), ra2 = up(ra, 4);
#pragma unroll
        for (int ks = 0; ks < D_KSUB; ++ks) {
            const int b = ks & 1;
            const bool last = ks + 1 == D_KSUB;
            const int ua = last ? ra1 : ra, ub = last ? rb1 : rb, rk = last ? 0 : ks + 1;
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const int i = m >> 1, j = m & 1;
                if (!last && m == 0) { read_b(ub, rk, b ^ 1, 0); read_b(ub, rk, b ^ 1, 1); }
                acc[i][j] = Half16<HT>::mfma(fa[i], fb[b][j], acc[i][j]);
                __builtin_amdgcn_sched_barrier(0);
                if (last && m == 1) {
                    __builtin_amdgcn_s_waitcnt(0x0074);   // vmcnt(4) lgkmcnt(0)
                    __builtin_amdgcn_s_barrier();
                    read_b(ub, rk, b ^ 1, 0);
                    read_b(ub, rk, b ^ 1, 1);
                }
                if (last && m >= 2 && m < 6) issue_b(next, next_kt, ra, m - 2);
                if (ks < 2 && (m == 2 || m == 6)) issue_a(next, next_kt, ra2, 2 * ks + (m >> 2));
                if (j == 1) read_a(ua, rk, i);           // row group i is done for this k-step: fetch the next one's
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };

    Src cur = make_src(tile);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int q = 0; q < 4; ++q) issue_a(cur, t, 2 * t, q);
#pragma unroll
        for (int q = 0; q < 4; ++q) issue_b(cur, t, 2 * t + 1, q);
    }
    __builtin_amdgcn_s_waitcnt(0x0F78);       // vmcnt(8): the first k-tile has landed
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < 4; ++i) read_a(0, 0, i);
    read_b(1, 0, 0, 0);
    read_b(1, 0, 0, 1);
    int ra = 0;

    const int rl = lane >> 4, cl = (lane & 15) * 4;

    while (true) {
        const int tm = tile / tiles_n, tn = tile - tm * tiles_n;
        li += n_slots;
        const int tile_next = tile_of(li);
        // no next tile: request this tile's first k-tile again (in bounds, never used)
        const Src nxt = make_src(tile_next >= 0 ? tile_next : tile);

        for (int kt = 0; kt < KT; ++kt) {
            // the last two k-tiles of a tile request the next tile's first two - by selecting the source, not by
            // branching: one straight-line loop body
            const bool wrap = kt + 2 >= KT;
            Src sel;
#pragma unroll
            for (int i = 0; i < 4; ++i) sel.a_off[i] = wrap ? nxt.a_off[i] : cur.a_off[i];
            sel.a_base = wrap ? nxt.a_base : cur.a_base;
            sel.b_base = wrap ? nxt.b_base : cur.b_base;
            ktile(ra, sel, wrap ? kt + 2 - KT : kt + 2);
            ra = up(ra, 2);
        }
        // here: the next tile's first k-tile is in LDS, the second on its way, fa / fb[0] hold the first fragments.  The unit
        // of this tile's last B operand stays free until the next tile's first k-tile refills it; each wave parks in the
        // part of it that it refills itself.
        float *ep = reinterpret_cast<float *>(lds + up(ra, 4) * D_OPB) + wave * 1024;

        // ---- epilogue.  In the accumulators a lane owns one column and sixteen rows of a 32x32 block
        // (register v: row 8 (v / 4) + 4 g + v % 4).  Sixteen rows x 64 columns at a time go through the
        // wave's parking slice and come back row-wise, four columns per lane, so that bias, GELU, the
        // residual and the stores move 8 or 16 bytes per lane in whole rows.  The slice has no padding:
        // rows with g = 1 keep their two 32-column halves swapped, which puts the 64 lanes of a write on
        // 64 different banks.  No branches: rows past M fall outside the buffer descriptor and are dropped.
        {
            const int row0 = tm * Q_BM + wm * 128, col0 = tn * Q_BN + wn * 64;
            int rows_left = M - row0;
            rows_left = rows_left < 0 ? 0 : (rows_left > 128 ? 128 : rows_left);
            OutT *cbase = C + (size_t)row0 * N + col0;
            const int n_bytes = rows_left > 0 ? ((rows_left - 1) * N + 64) * (int)sizeof(OutT) : 0;
            const rsrc_t c_rs = __builtin_amdgcn_make_buffer_rsrc(cbase, 0, n_bytes, 0x00020000);
            // The lane part of every address is one register, made opaque per tile: left alone, the compiler
            // moves the 32 row offsets of a tile out of the tile loop and keeps them in registers it does not have.
            // The row-group part of an address is wave-uniform and travels as the scalar offset of the access.
            int lane_off = (rl * N + cl) * (int)sizeof(OutT);
            asm volatile("" : "+v"(lane_off));
            const int row_step = N * (int)sizeof(OutT);
            const f32x4 bv4 = *reinterpret_cast<const f32x4 *>(bias + col0 + cl);
#pragma unroll
            for (int n = 0; n < 8; ++n) {
                const int i = n >> 1, hh = n & 1;
                f32x4 val[4], res[4];
                if constexpr (EPI == EPI_BIAS_RESIDUAL) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int r0 = 32 * i + 16 * hh + 4 * q;
                        res[q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(c_rs, r0 + rl < rows_left ? lane_off : kOutside, r0 * row_step, 0));
                    }
                }
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int vv = 0; vv < 8; ++vv)
                        ep[(8 * (vv >> 2) + 4 * g + (vv & 3)) * 64 + 32 * (j ^ g) + l32] = acc[i][j][8 * hh + vv];
                asm volatile("" ::: "memory");       // a wave's LDS operations execute in order: no wait, only the order
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
                    const int v_off = r0 + rl < rows_left ? lane_off : kOutside;   // rows past M: an offset no buffer holds
                    f32x4 o = val[q] + bv4;
                    if constexpr (EPI == EPI_BIAS_GELU) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = gelu_erf_h16(o[e]);
                    }
                    if constexpr (OUT_F32) {
                        if constexpr (EPI == EPI_BIAS_RESIDUAL) o += res[q];
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, o), c_rs, v_off, s_off, 0);
                    } else {
                        v4 o4;
#pragma unroll
                        for (int e = 0; e < 4; ++e) o4[e] = from_f32<HT>(o[e]);
                        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i32x2, o4), c_rs, v_off, s_off, 0);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): this wave has read back what it parked
        if (tile_next < 0) break;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
        tile = tile_next;
        cur = nxt;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);       // the loads of the unused last requests have landed before the LDS goes away
}

int p8_cus() {
    static std::atomic<int> cus{0};
    int c = cus.load(std::memory_order_acquire);
    if (c == 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        c = (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) ? prop.multiProcessorCount : 256;
        if (c < 8) c = 8;
        cus.store(c, std::memory_order_release);
    }
    return c;
}

}  // namespace

bool gemm_p8_applicable(int M, int N, int K) {
    return M >= 1 && N >= 256 && N % 256 == 0 && K >= 128 && K % 64 == 0 && (long long)N * 4 * 128 < (1ll << 31) &&
           (long long)((M + 255) / 256) * (N / 256) < (1ll << 30);
}

template <typename HT, typename OutT, int EPI>
static void launch_p8_one(const HT *A, const HT *Bt, const float *bias, OutT *C, int M, int N, int K, hipStream_t s) {
    const int tiles_m = (M + Q_BM - 1) / Q_BM, tiles_n = N / Q_BN;
    const int per_xcd = ((tiles_m + 7) / 8) * tiles_n;      // tiles of the XCD with the most row panels
    const int slots = per_xcd < p8_cus() / 8 ? per_xcd : p8_cus() / 8;
    auto kern = gemm_h16_p8_kernel<HT, OutT, EPI>;
    static std::atomic<bool> attr_set{false};   // callers may come from several host threads
    if (!attr_set.load(std::memory_order_acquire)) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, D_LDS);
        attr_set.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3(8 * slots), dim3(512), D_LDS, s, A, Bt, bias, C, M, N, K, tiles_m, tiles_n, Q_CB);
}

template <typename HT, typename OutT>
void launch_gemm_p8(const HT *A, const HT *Bt, const float *bias, OutT *C, int M, int N, int K, Epi epi, hipStream_t s) {
    if constexpr (sizeof(OutT) == 4) {
        if (epi == EPI_BIAS_RESIDUAL) launch_p8_one<HT, float, EPI_BIAS_RESIDUAL>(A, Bt, bias, C, M, N, K, s);
        else launch_p8_one<HT, float, EPI_BIAS>(A, Bt, bias, C, M, N, K, s);
    } else {
        if (epi == EPI_BIAS_GELU) launch_p8_one<HT, HT, EPI_BIAS_GELU>(A, Bt, bias, C, M, N, K, s);
        else launch_p8_one<HT, HT, EPI_BIAS>(A, Bt, bias, C, M, N, K, s);
    }
}
template void launch_gemm_p8<bf16, bf16>(const bf16 *, const bf16 *, const float *, bf16 *, int, int, int, Epi, hipStream_t);
template void launch_gemm_p8<bf16, float>(const bf16 *, const bf16 *, const float *, float *, int, int, int, Epi, hipStream_t);
template void launch_gemm_p8<f16, f16>(const f16 *, const f16 *, const float *, f16 *, int, int, int, Epi, hipStream_t);
template void launch_gemm_p8<f16, float>(const f16 *, const f16 *, const float *, float *, int, int, int, Epi, hipStream_t);

}  // namespace sjd

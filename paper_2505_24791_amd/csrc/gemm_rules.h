// Which launches of a 16-bit projection the persistent kernels take.  Plain C++ beside the kernels, so that the arithmetic can be
// checked without a device.
#pragma once

namespace sjd {

constexpr int kXcds = 8, kCusPerXcd = 32;
constexpr int kP8Tile = 256;                    // gemm_p8.hip: tiles of 256 x 256, one workgroup per CU
constexpr int kDuoRows = 128, kDuoCols = 256;   // gemm_duo.hip: tiles of 128 x 256, two workgroups per CU

// Both kernels deal whole row panels to the XCDs: tiles of the one with the most of them.
inline long long tiles_of_fullest_xcd(int M, int N, int rows, int cols) {
    const long long panels = ((long long)M + rows - 1) / rows;
    return (panels + kXcds - 1) / kXcds * (((long long)N + cols - 1) / cols);
}

inline bool gemm_p8_one_round(int M, int N) { return tiles_of_fullest_xcd(M, N, kP8Tile, kP8Tile) <= kCusPerXcd; }

// MLP-input projection with GELU on gemm_duo.hip: from one tile per CU on, but not where gemm_p8.hip is through in one round, unless
// every CU gets exactly one tile.  In between some CUs have two workgroups and the others one, with nothing to hide GELU behind, and
// tiles of half the height pull a layer's weights into an XCD's L2 twice as often; on weights that are still there from the launch before the
// kernel wins all the same (3000 x 3072 x 768, 288 tiles: 28.1 -> 27.2 us), in a pass of several layers it does not.  Microseconds a pass, the other
// kernels -> this one:
//   one round of gemm_p8.hip: width 768, 8 layers, 288 tiles 1018 -> 1080, 384 tiles 966 -> 1003; width 1024, 8 layers, 288 / 336 / 384 / 448 tiles 1052 ->
//     1123, 1093 -> 1154, 1141 -> 1217, 1252 -> 1278; width 512, 8 layers, 448 tiles 850 -> 868; width 256, 6 layers, 436 tiles 535 -> 545; width 640, 6 layers,
//     260 tiles 692 -> 714;
//   two rounds, or 128 x 128 tiles: width 768, 396 tiles 1093 -> 1021, 804 tiles 1795 -> 1797; width 1024, 528 tiles 1964 -> 1840; width 512, 4 layers, 528
//     tiles 618 -> 587; width 256, 516 tiles 696 -> 650;
//   one tile for every CU (256): width 1024 955 -> 932, width 512, 4 layers 356 -> 347.  Below: 1024 x 3072 x 768 (96 tiles) 14.6 -> 16.2 us alone.
inline bool gemm_duo_applicable(int M, int N, int K) {
    if (N < 256 || N % 256 || K < 256 || K % 128 || (long long)N * K * 2 >= (1ll << 31) || (long long)N * 2 * 128 >= (1ll << 31)) return false;
    const long long tiles = ((long long)M + kDuoRows - 1) / kDuoRows * (N / kDuoCols);
    if (tiles < kXcds * kCusPerXcd || tiles >= (1ll << 30)) return false;
    return tiles_of_fullest_xcd(M, N, kDuoRows, kDuoCols) <= kCusPerXcd || !gemm_p8_one_round(M, N);
}

// Deep k-loops that the persistent kernel does not cover: one 256x256 tile to a CU (gemm_h16_dma_kernel) or two workgroups with 128x128
// rings.  A full round of large tiles takes as long as 1.68 rounds of two small ones a CU (1.78 with GELU, which the ring's other workgroup hides):
// 8192 x 2000 x 4096 117.3 us against 145.2, 8192 x 2000 x 1024 37.0 / 44.1, 32768 x 1000 x 4096 (two rounds) 244.7 / 306.7, its GELU 259 / 316.  A last
// round that is partly empty takes half of one or more: 24000 x 600 x 4096 (1.1 rounds) 187.7 / 138.1, 24000 x 1000 x 4096 (1.5) 206.7 / 214.1, with GELU
// 221.6 / 220.4, 24000 x 1100 x 4096 (1.8) 222.7 / 251.2, 12288 x 2688 x 896 (2.1) 87.5 / 77.1.  In a pass: MLP output of width 896, 32768 rows 240 / 273, of 960, 49152 rows
// 378 / 463; QKV of 896, 16640 rows 100 / 111.
inline bool gemm_dma_before_ring(int M, int N, bool gelu) {
    const long long large = (((long long)M + 255) / 256) * (((long long)N + 255) / 256), small = (((long long)M + 127) / 128) * (((long long)N + 127) / 128);
    if (M < 256 || N < 256 || large < kXcds * kCusPerXcd) return false;
    auto rounds = [](double r, double started, double filled) {
        const double whole = (double)(long long)r;
        return whole + (r > whole ? started + filled * (r - whole) : 0.0);
    };
    return (gelu ? 1.78 : 1.68) * rounds(large / 256.0, 0.5, 0.45) < rounds(small / 512.0, 0.25, 0.75);
}

}  // namespace sjd

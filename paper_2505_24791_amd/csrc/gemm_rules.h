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

}  // namespace sjd

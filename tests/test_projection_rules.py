"""The rules that give a 16-bit projection to one of the persistent kernels (csrc/gemm_rules.h), compiled for the host."""
import pytest


def test_tiles_of_the_fullest_xcd_are_those_that_the_kernels_deal(launch_rules):
    for rows in (1, 127, 128, 129, 1000, 3000, 4607, 32768):
        for bm in (128, 256):
            panels = -(-rows // bm)
            dealt = [(x + 1) * panels // 8 - x * panels // 8 for x in range(8)]      # as in gemm_p8.hip and gemm_duo.hip
            assert launch_rules.fullest(rows, 3072, bm, 256) == max(dealt) * 12


@pytest.mark.parametrize("N,K", [(1024, 256), (1536, 384), (2048, 512), (2560, 640), (3072, 768), (4096, 1024), (5120, 1280)])
def test_two_workgroups_per_cu_only_where_one_per_cu_needs_a_second_round(launch_rules, N, K):
    """A launch that the 256 x 256 tiles of gemm_p8.hip finish in one round stays there (a pass of width 1024 and 384 tiles: 1141 us
    instead of 1217), unless every CU gets exactly one tile of this kernel."""
    taken = 0
    for panels in range(1, 400):
        for M in (128 * panels - 127, 128 * panels):
            tiles = panels * N // 256
            one_round = -(-(-(-M // 256)) // 8) * N // 256 <= 32
            one_each = tiles == 256 and -(-panels // 8) * N // 256 <= 32
            assert launch_rules.duo(M, N, K) == (tiles >= 256 and (one_each or not one_round)), M
            taken += launch_rules.duo(M, N, K)
    assert taken > 100


def test_launches_that_the_kernel_does_not_cover(launch_rules):
    assert launch_rules.duo(32768, 4096, 1024)
    for M, N, K in [(32768, 4096 + 128, 1024), (32768, 4096, 1024 + 64), (32768, 1024, 128), (32768, 1 << 20, 1024), (1, 4096, 1024)]:
        assert not launch_rules.duo(M, N, K), (M, N, K)


def test_large_tiles_where_their_last_round_is_full(launch_rules):
    """Deep k-loops with N not a multiple of 256: 256x256 tiles where they beat two 128x128 rings a CU (microseconds beside the rule)."""
    dma = launch_rules.dma_before_ring
    for m, n in ((8192, 2000), (32768, 1000), (24000, 2000), (24576, 1152), (8192, 3456), (12288, 3456), (32768, 896), (16640, 2688), (24000, 1100), (49152, 960)):
        assert dma(m, n, 0), (m, n)
    for m, n in ((24000, 600), (12288, 2688), (16640, 1000), (16640, 1100), (6000, 2688), (24576, 896)):
        assert not dma(m, n, 0) and not dma(m, n, 1), (m, n)
    assert dma(24000, 1000, 0) and not dma(24000, 1000, 1)         # one and a half rounds: GELU hides better beside the rings
    assert not dma(255, 65536, 0) and not dma(65536, 255, 0) and not dma(4096, 3840, 0)
    assert dma(4096, 4000, 0)                                       # one tile for every CU

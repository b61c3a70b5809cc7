"""The automatic choice between the kernels, where measured times say clearly which one it should be: random problems of sweep.py
--tiles, each with the times (us) of the second kernel (tiles "-rb") and of the fourth (160x256/2x4w/3s, 128x256/2x4w/3s)."""
import pytest

import paper_2508_16584_amd as gg
from paper_2508_16584_amd.binding import load_library

FOURTH = ("160x256/2x4w/3s", "128x256/2x4w/3s")


@pytest.mark.parametrize("G,M,N,K,second,fourth", [
    (2, 28849, 5248, 640, 148.7, 116.6), (3, 30129, 5504, 640, 157.9, 127.7), (3, 25644, 5888, 640, 145.5, 121.6),       # 5 K blocks
    (11, 2715, 7424, 6784, 234.6, 189.2), (34, 21212, 4224, 2176, 249.1, 217.7), (1, 13083, 1536, 6016, 135.0, 116.6),   # 53, 17, 47
    (7, 3123, 5760, 640, 27.3, 20.6), (1, 1289, 4480, 5504, 55.4, 44.2)])
def test_an_odd_number_of_k_blocks_costs_the_second_kernel(G, M, N, K, second, fourth):
    assert K // 128 % 2 == 1 and fourth < 0.9 * second
    assert gg.variant_name(gg.auto_variant(G, M, N, K)) in FOURTH


def test_the_odd_number_is_the_only_step_along_k():
    """The odd number's cost is the only step in K: where the second kernel is chosen with an odd number of K blocks, it is with
    both even neighbours."""
    second = lambda G, M, N, kb: gg.variant_name(gg.auto_variant(G, M, N, 128 * kb)).endswith("-rb")
    seen = 0
    for G, M, N in [(8, 3001, 4096), (8, 8192, 4096), (4, 12000, 2048), (16, 16384, 7168), (32, 16384, 7168), (2, 6000, 8192)]:
        for kb in range(5, 64, 2):
            if second(G, M, N, kb):
                seen += 1
                assert second(G, M, N, kb - 1) and second(G, M, N, kb + 1), (G, M, N, kb)
    assert seen > 20


@pytest.mark.parametrize("G,M,N,K,small,narrow", [(4, 8090, 336, 7168, 71.5, 43.9), (5, 12196, 184, 5888, 57.9, 35.3), (2, 8029, 336, 3072, 31.4, 22.7),
                                                  (22, 6786, 320, 5632, 44.2, 34.8), (18, 1952, 1120, 7808, 60.9, 48.8)])
def test_ragged_n_that_a_256_wide_tile_would_mostly_waste(G, M, N, K, small, narrow):
    """... and here those of the 64 x 128 and the 128 x 128 tile."""
    assert narrow < 0.9 * small and gg.variant_name(gg.auto_variant(G, M, N, K)) == "128x128/2x4w/4s"


@pytest.mark.parametrize("G,M,N,K", [(64, 2048, 4096, 7168), (256, 32768, 4096, 7168), (8, 8192, 4096, 7168), (40, 300, 1024, 2048), (12, 900, 768, 640), (3, 5, 512, 512)])
def test_padded_problems_go_by_the_rows_that_their_groups_are_expected_to_hold(G, M, N, K):
    cap = gg.padded_rows_cap(G, M)
    assert gg.auto_variant_padded(G, cap, N, K) == gg.auto_variant(G, cap - 64 * G, N, K)


@pytest.mark.parametrize("G,M,N,K,third,fifth", [(1, 16, 5888, 4224, 22.0, 8.5), (4, 65, 640, 5120, 14.5, 6.5), (37, 1, 1280, 7808, 19.1, 7.3), (13, 2, 768, 2176, 8.6, 4.3)])
def test_chains_of_k_blocks_on_few_tiles(G, M, N, K, third, fifth):
    """... and here those of the third and the fifth kernel."""
    assert fifth < 0.7 * third and gg.variant_name(gg.auto_variant(G, M, N, K)) in ("16x16/8x1w/3s", "16x32/4x1w/3s", "16x32/4x1w/2s")


@pytest.mark.parametrize("G,M,N,K,other,fifth", [(49, 4, 7168, 3328, 18.4, 22.8), (221, 13, 2304, 3072, 18.3, 22.5), (13, 6, 5376, 2560, 16.1, 18.5),
                                                 (4, 43, 6376, 3968, 22.8, 25.9), (8, 27, 3480, 4912, 25.7, 27.7), (9, 151, 1920, 512, 7.0, 7.4)])
def test_a_little_more_than_one_round_of_chains(G, M, N, K, other, fifth):
    """The last tiles take as long as all others: the 16 x 32 tiles are taken up to one round (here: with the best other kernel's time)."""
    assert other < fifth and gg.variant_name(gg.gemm_route(G, M, N, K)) not in ("16x32/4x1w/3s", "16x32/4x1w/2s")


@pytest.mark.parametrize("G,M,N,K", [(16034763, 2, 4288, 128), (1 << 24, 3, 4096, 256), (1 << 30, 1, 520, 400)])
def test_groups_without_rows_are_no_tiles_of_the_fifth_kernel(G, M, N, K):
    """It has a workgroup for every tile there may be, and no more groups hold rows than there are rows."""
    assert gg.variant_name(gg.gemm_route(G, M, N, K)) in ("16x16/8x1w/3s", "16x32/4x1w/3s", "16x32/4x1w/2s")


def test_the_route_is_the_named_choice_where_there_is_one():
    for G, M, N, K in [(4, 300, 640, 640), (37, 1, 1280, 7808), (8, 8192, 4096, 7168), (64, 2048, 4096, 7168), (256, 128, 2048, 2048), (3, 5, 512, 512)]:
        assert gg.gemm_route(G, M, N, K) == gg.gemm_route(G, M, N, K, sa_kmajor=True) == gg.auto_variant(G, M, N, K)
        cap = gg.padded_rows_cap(G, M)
        assert gg.gemm_route(G, cap, N, K, padded=True) == gg.auto_variant_padded(G, cap, N, K)
    for G, M, N, K in [(4, 8, 12, 512), (4, 8, 256, 24), (-1, 8, 256, 512), (4, 8, (1 << 21) + 8, 512)]:
        with pytest.raises(ValueError):
            gg.gemm_route(G, M, N, K)
    with pytest.raises(ValueError):
        gg.gemm_route(4, 1 << 24, 256, 1 << 20, sa_kmajor=True)
    assert load_library().gg_fp8_gemm_route(4, 8, 256, 512, 8) == -3


@pytest.mark.parametrize("G,M,N,K", [(5, 20, 264, 400), (3, 7, 8, 512), (4, 30, 136, 2000)])
def test_the_route_names_the_fifth_kernel_on_ragged_sizes_too(G, M, N, K):
    assert gg.gemm_route(G, M, N, K) >= 26 > gg.auto_variant(G, M, N, K)

"""How the weight-gradient call runs (gg_fp8_wgrad_route), as far as it must not depend on sizes that were measured."""
import numpy as np
import pytest
import torch

import bench
import paper_2508_16584_amd as gg
from workloads import CONFIGS, group_sizes


@pytest.mark.parametrize("out_bf16", [False, True])
def test_scales_between_two_16_byte_pieces_stay_with_the_narrow_tiles(out_bf16):
    """The 256 x 256 tiles fetch 16 bytes of scales per lane, the narrow ones four: only those take any float tensor."""
    G, M, N, K = 8, 32768, 8192, 8192
    flat = torch.empty(64)
    flat = flat[-(flat.data_ptr() // 4) % 4:]
    assert "square" in gg.wgrad_route(G, M, N, K, out_bf16, flat, flat[4:])
    for first in (1, 2, 3):
        assert not gg.wgrad_route(G, M, N, K, out_bf16, flat[first:], flat)
        assert not gg.wgrad_route(G, M, N, K, out_bf16, flat, flat[first:])


# Random problems with the measured times (us) of the narrow and the square tiles: skewed groups in few rounds over the workgroups, or
# groups so short that the stores bound them; then even or long ones.
@pytest.mark.parametrize("G,M,N,K,out_bf16,narrow,square", [
    (214, 28208, 768, 1280, True, 165.1, 213.6), (23, 7552, 4608, 1792, True, 136.5, 169.5), (101, 24000, 2304, 768, True, 165.6, 205.3),
    (182, 27072, 2048, 512, True, 149.4, 175.9), (125, 28112, 1792, 768, False, 174.1, 204.1), (4, 960, 8192, 8192, False, 211.9, 246.9),
    (8, 1680, 8192, 8192, False, 427.9, 498.5), (43, 12976, 2560, 1792, True, 170.5, 198.2), (127, 32688, 1280, 1280, False, 225.6, 260.1),
    (45, 12992, 768, 5120, True, 145.0, 166.0), (26, 11408, 4864, 1536, False, 225.6, 241.9),
    (99, 20992, 1024, 4864, False, 592.0, 411.3), (55, 31168, 3328, 2048, False, 645.5, 500.4), (17, 28432, 2816, 3584, True, 479.4, 406.7),
    (17, 12048, 1792, 7424, False, 424.4, 331.9), (4, 6768, 8192, 6144, True, 535.3, 437.8), (202, 28432, 1280, 4608, True, 913.3, 767.5),
    (13, 13744, 3328, 6400, False, 647.1, 538.2), (37, 19312, 4096, 4096, False, 963.0, 812.7)])
def test_tiles_where_measured_times_say_which(G, M, N, K, out_bf16, narrow, square):
    assert ("square" in gg.wgrad_route(G, M, N, K, out_bf16)) == (square < narrow)


# Operands of 140 to 192 MB with the measured times (us) of the square tiles without and with the operands brought in ahead
@pytest.mark.parametrize("G,M,N,K,out_bf16,plain,ahead", [
    (17, 28432, 2816, 3584, True, 393.2, 406.7), (10, 16000, 2304, 7424, True, 431.2, 449.4), (9, 21744, 2560, 6656, False, 548.6, 577.8),
    (18, 22544, 1536, 5632, True, 312.3, 334.5), (19, 24112, 6400, 1536, False, 412.8, 423.4), (26, 18016, 1280, 7680, False, 396.5, 408.1),
    (23, 26240, 2816, 2816, False, 336.5, 348.7), (19, 23040, 1792, 5632, False, 365.3, 378.7),
    (110, 30480, 4096, 1024, False, 675.1, 596.0), (191, 29968, 768, 4608, False, 683.1, 610.5), (109, 23312, 5888, 2048, True, 1096.5, 983.9),
    (93, 29680, 1280, 5376, False, 786.1, 720.9), (76, 27104, 5888, 1280, False, 714.0, 658.8)])
def test_operands_ahead_where_measured_times_say_so(G, M, N, K, out_bf16, plain, ahead):
    way = gg.wgrad_route(G, M, N, K, out_bf16)
    assert "square" in way and ("ahead" in way) == (ahead < plain)


# Few outputs that meet many tokens, and others: measured times (us) of the narrow tiles and of those with the blocks dealt to the waves
@pytest.mark.parametrize("G,M,N,K,out_bf16,narrow,chain", [
    (2, 11472, 256, 768, False, 96.2, 25.9), (1, 944, 1280, 512, False, 24.1, 6.9), (5, 272, 768, 256, False, 11.7, 4.1), (1, 5520, 896, 1024, True, 90.8, 25.5),
    (2, 2288, 896, 3584, True, 28.8, 42.5), (20, 2288, 640, 512, True, 13.7, 20.2), (220, 64, 384, 512, False, 36.5, 55.2), (7, 112, 256, 2048, True, 6.6, 10.1),
    (5, 1264, 768, 1280, False, 14.7, 17.8)])
def test_blocks_dealt_to_waves_where_measured_times_say_so(G, M, N, K, out_bf16, narrow, chain):
    assert ("chain" in gg.wgrad_route(G, M, N, K, out_bf16)) == (chain < narrow)


# Narrow tiles, whole and halved: measured times (us)
@pytest.mark.parametrize("G,M,N,K,out_bf16,whole,half", [
    (19, 400, 256, 512, True, 7.6, 5.8), (7, 160, 256, 2048, False, 8.3, 6.4), (2, 5120, 640, 2304, True, 47.5, 42.3), (24, 384, 768, 256, True, 7.6, 6.7),
    (2, 992, 1280, 2816, False, 20.4, 16.1), (7, 272, 640, 3840, True, 15.9, 13.7), (2, 6880, 8064, 1024, True, 78.3, 91.1),
    (2, 5184, 5888, 4864, True, 203.9, 232.2), (14, 2128, 256, 3584, True, 20.6, 22.1), (96, 64, 384, 3328, True, 48.7, 53.3)])
def test_halved_tiles_where_measured_times_say_so(G, M, N, K, out_bf16, whole, half):
    assert ("half" in gg.wgrad_route(G, M, N, K, out_bf16)) == (half < whole)


# The same where K is a multiple of 2048 and the halves are more than a round
@pytest.mark.parametrize("G,M,N,K,out_bf16,whole,half", [
    (13, 608, 1024, 2048, False, 24.4, 32.6), (8, 848, 1024, 2048, False, 19.1, 22.1), (8, 272, 1024, 4096, False, 29.2, 32.4), (4, 320, 896, 4096, True, 13.6, 14.9),
    (6, 704, 1280, 4096, True, 24.0, 25.6), (59, 7472, 256, 2048, False, 32.6, 34.6)])
def test_rows_of_whole_4_kb_are_not_halved(G, M, N, K, out_bf16, whole, half):
    assert whole < half and "half" not in gg.wgrad_route(G, M, N, K, out_bf16)
    assert "half" in gg.wgrad_route(G, M, N, K - 256, out_bf16) and "half" in gg.wgrad_route(1, 128, 768, K, out_bf16)


@pytest.mark.parametrize("workload,kernel", [("gate_up", "gg_wgrad_sq_kernel"), ("down", "gg_wgrad_sq_kernel"), ("decode", "gg_wgrad_kernel")])
@pytest.mark.parametrize("out_bf16", [False, True])
def test_the_benchmark_names_the_kernel_that_runs(workload, kernel, out_bf16):
    c = CONFIGS[workload]
    assert bench.wgrad_kernel(c.G, int(np.sum(group_sizes(c, c.seed))), c.N, c.K, out_bf16) == kernel


def test_what_the_call_refuses_has_no_route():
    for G, M, N, K in [(-1, 16, 256, 256), (4, 17, 256, 256), (4, 16, 200, 256), (4, 16, 256, 128), (4, 1 << 24, 256, 256), (4, 16, 256, 1 << 21)]:
        with pytest.raises(ValueError):
            gg.wgrad_route(G, M, N, K)
    assert gg.wgrad_route(0, 16, 256, 256) == set()

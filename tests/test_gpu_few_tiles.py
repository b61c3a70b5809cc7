"""The fifth kernel (K blocks dealt to the waves of a workgroup) where it can go wrong: numbers of K blocks around what a round of
its waves, one slot and both slots take, rows around its tiles, ragged N and K (which only the automatic choice runs on it), a
K loop that does not start at block 0, both orders of the scales, both outputs, more groups than one lookup holds."""
import numpy as np
import pytest
import torch

import paper_2508_16584_amd as gg
from gg_testlib import assert_parity, bits_of
from oracle import gg_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TILES = ("16x16/8x1w/3s", "16x32/4x1w/3s", "16x32/4x1w/2s")
FIRST = 2                                  # 128 x 128 tile of the first kernel: any shape


def problem(sizes, N, K, seed):
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    M, G, KB, NB = int(off[-1]), len(sizes), -(-K // 128), -(-N // 128)
    A = rng.integers(0, 0x70, (M, K), dtype=np.uint8) | (rng.integers(0, 2, (M, K), dtype=np.uint8) << 7)
    B = rng.integers(0, 0x48, (G, N, K), dtype=np.uint8) | (rng.integers(0, 2, (G, N, K), dtype=np.uint8) << 7)
    SA = rng.uniform(0.5, 2.0, (M, KB)).astype(np.float32)
    SB = rng.uniform(0.5, 2.0, (G, NB, KB)).astype(np.float32)
    return A, SA, B, SB, off


def check(sizes, N, K, seed, tiles=TILES):
    host = problem(sizes, N, K, seed)
    dA, dSA, dB, dSB, doff = (torch.from_numpy(x).to(DEV) for x in host)
    want = gg.grouped_gemm(dA, dSA, dB, dSB, doff, variant=FIRST)
    assert_parity(bits_of(want), orc.grouped_gemm(*host, with_abs_sum=True), empirical=False, what=f"{sizes} N={N} K={K}")
    SAk = dSA.t().contiguous()
    for v in [-1] + [u for u in range(gg.num_variants()) if gg.variant_name(u) in tiles]:
        for scales, km in ((dSA, False), (SAk, True)):
            C = torch.full((want.shape[0] + 2, N), 0x7FC1, dtype=torch.int16, device=DEV).view(torch.bfloat16)
            gg.grouped_gemm(dA, scales, dB, dSB, doff, C=C[:-2], variant=v, sa_kmajor=km)
            assert torch.equal(C[:-2].view(torch.int16), want.view(torch.int16)), (v, km)
            assert (C[-2:].view(torch.int16) == 0x7FC1).all(), "wrote past the last row"
    h = gg.grouped_gemm(dA, dSA, dB, dSB, doff, out_dtype=torch.float16)
    assert torch.equal(h.view(torch.int16), gg.grouped_gemm(dA, dSA, dB, dSB, doff, variant=FIRST, out_dtype=torch.float16).view(torch.int16))


@pytest.mark.parametrize("blocks", [1, 3, 4, 5, 7, 8, 9, 12, 13, 16, 17, 24, 25, 33])
def test_k_blocks_around_rounds_and_slots(blocks):
    assert gg.variant_name(gg.auto_variant(5, 36, 256, 128 * blocks)) in TILES
    check([1, 15, 0, 3, 17], 256, 128 * blocks, blocks)


@pytest.mark.parametrize("sizes", [[1], [16], [17], [33, 1], [0, 15, 0, 16, 1]])
def test_rows_around_tiles(sizes):
    check(sizes, 384, 640, sum(sizes))


@pytest.mark.parametrize("N,K", [(8, 512), (264, 512), (280, 1040), (256, 16), (136, 2000), (504, 400)])
def test_ragged_shapes_of_the_automatic_choice(N, K):
    check([5, 0, 20, 2], N, K, N + K, tiles=())


@pytest.mark.parametrize("tile,sizes,N,K", [
    # N no multiple of the tile's columns, of 16 and of 32; short last K blocks in the first round and after one, two and more refills
    (0, [14], 8, 560), (0, [0, 29, 1, 15], 24, 1136), (0, [3, 17], 40, 2080), (0, [2, 0, 31], 264, 3152), (0, [5, 12], 136, 4368), (0, [20], 40, 3840),
    (1, [114], 520, 592), (1, [60, 0, 41, 5], 472, 1120), (1, [99], 712, 1920), (1, [17, 33, 1, 48], 664, 1712), (1, [107], 688, 3344), (1, [111], 552, 640),
    (2, [11], 24, 32), (2, [40, 0, 70, 8], 1192, 544), (2, [5, 33, 64, 16], 1240, 1136), (2, [17, 0, 33, 16, 1, 49, 1], 1192, 1696),
    (2, [3, 30, 0, 16, 17, 1, 33, 10, 7], 1192, 2064), (2, [17, 0, 33, 17, 1, 49, 1], 1224, 1920)])
def test_ragged_shapes_on_every_tile(tile, sizes, N, K):
    """Only the automatic choice runs these sizes on the fifth kernel: on the tile that the route names."""
    G, M = len(sizes), sum(sizes)
    assert gg.variant_name(gg.gemm_route(G, M, N, K)) == gg.variant_name(gg.gemm_route(G, M, N, K, sa_kmajor=True)) == TILES[tile]
    check(sizes, N, K, N + K, tiles=())


def test_rotated_k_loop():
    check([3, 18], 768, 4096, 1)


def test_more_groups_than_one_lookup_holds():
    sizes = [0] * 300
    for g in (0, 63, 64, 200, 255, 256, 270, 299):
        sizes[g] = 1 + g % 3
    check(sizes, 256, 384, 2)


def test_groups_past_the_first_256_are_found_64_at_a_time():
    sizes = [0] * 700
    for g in (3, 255, 256, 257, 300, 319, 320, 383, 384, 447, 513, 640, 698, 699):
        sizes[g] = 1 + g % 18
    assert gg.variant_name(gg.auto_variant(700, sum(sizes), 128, 256)) in TILES
    check(sizes, 128, 256, 4)
    check(sizes[:513] + [0] * 187, 128, 256, 5)         # the last rows before the last groups


def test_a_lookup_costs_little_however_many_groups_there_are():
    """Few rows: 5 us with 256 groups, 13 with 2048 (191 where every workgroup walks the groups one by one)."""
    def us(G, N=256, K=512, M=8, launches=20):
        A, SA = torch.zeros(M, K, dtype=torch.uint8, device=DEV), torch.ones(M, K // 128, device=DEV)
        B, SB = torch.zeros(G, N, K, dtype=torch.uint8, device=DEV), torch.ones(G, N // 128, K // 128, device=DEV)
        off = torch.zeros(G + 1, dtype=torch.int32)
        off[G - M + 1:] = torch.arange(1, M + 1)        # a row for each of the last groups
        off, C = off.to(DEV), torch.empty(M, N, dtype=torch.bfloat16, device=DEV)
        assert gg.variant_name(gg.auto_variant(G, M, N, K)) in TILES
        gg.grouped_gemm(A, SA, B, SB, off, C=C)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(launches):
                gg.grouped_gemm(A, SA, B, SB, off, C=C)
        begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        times = []
        for _ in range(6):
            begin.record()
            graph.replay()
            end.record()
            torch.cuda.synchronize()
            times.append(begin.elapsed_time(end) / launches * 1e3)
        return sorted(times)[2]
    few, many = us(256), us(2048)
    assert many < 6 * few, (few, many)


def test_ragged_shapes_are_refused_by_name():
    dev = tuple(torch.from_numpy(x).to(DEV) for x in problem([4, 2], 264, 400, 3))
    for v in [u for u in range(gg.num_variants()) if gg.variant_name(u) in TILES]:
        with pytest.raises(gg.GGError) as e:
            gg.grouped_gemm(*dev, variant=v)
        assert e.value.status == 3
    assert gg.variant_name(gg.auto_variant(2, 6, 264, 400)) not in TILES        # ... and not named by the choice

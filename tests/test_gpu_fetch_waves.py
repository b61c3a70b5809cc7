"""The kernel whose waves either fetch or multiply (tiles 160x256 and 128x256): the same bits as the first kernel's 128x128
tile, which takes every shape, where its tiles, its K loop and its chunks of scales end, and at every height it chooses."""
import math

import numpy as np
import pytest
import torch

import paper_2508_16584_amd as gg
from gg_testlib import assert_parity, bits_of
from oracle import gg_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
OTHER = 2


def problem(sizes, N, K, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    M, G, KB, NB = int(sum(sizes)), len(sizes), -(-K // 128), -(-N // 128)
    A = torch.randint(0, 256, (M, K), generator=gen, device=DEV, dtype=torch.uint8) & 0xBF       # no NaN codes
    B = torch.randint(0, 256, (G, N, K), generator=gen, device=DEV, dtype=torch.uint8) & 0xBF
    SA = torch.rand((M, KB), generator=gen, device=DEV) + 0.5
    SB = torch.rand((G, NB, KB), generator=gen, device=DEV) + 0.5
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)).to(DEV)
    return A, SA, B, SB, off


def check(dev, K, what):
    A, SA, B, SB, off = dev
    SAk = SA.t().contiguous()
    for dt in (torch.bfloat16, torch.float16):
        want = gg.grouped_gemm(A, SA, B, SB, off, variant=OTHER, out_dtype=dt)
        for v in (-1, 0, 3):
            for km in (False, True):
                got = gg.grouped_gemm(A, SAk if km else SA, B, SB, off, variant=v, sa_kmajor=km, out_dtype=dt)
                assert torch.equal(got.view(torch.int16), want.view(torch.int16)), f"{what}: variant {v} kmajor {km} {dt}"


# heights of 1 to 5 steps of 32 rows, full and one row more or less; groups of two and three tiles of equal height; one,
# two, ... K blocks (chunks of eight, tiles shorter than the ring), a short last K block, partial tiles along N
@pytest.mark.parametrize("K", [128, 256, 384, 512, 1024, 1040, 1152, 2176, 4096])
@pytest.mark.parametrize("N", [256, 264, 320, 1152])
def test_tile_heights_and_k_blocks(N, K):
    sizes = [1, 31, 32, 0, 33, 159, 160, 161, 0, 16, 17, 127, 129, 320, 321, 481]
    check(problem(sizes, N, K, N + K), K, f"N={N} K={K}")


@pytest.mark.parametrize("sizes", [[128] * 40, [97, 30, 200] * 60, [3] * 300 + [170], [0] * 70 + [90] + [0] * 250 + [150]])
def test_many_tiles_and_many_groups(sizes):
    """Launches of several rounds; more groups than one index holds."""
    N, K = 2048, 640
    check(problem(sizes, N, K, len(sizes)), K, f"{len(sizes)} groups")


def chosen_height(sizes, N):
    """The rule of the kernel (pc_height), written out again: another height gives the same bits, so this only says which heights
    the cases below are meant to reach."""
    columns = -(-N // 256)
    grid = min(256, (sum(sizes) // 32 + len(sizes)) * columns)
    grid -= grid % 8 if grid >= 8 else 0
    tiles = {bm: sum(-(-s // bm) for s in sizes) for bm in (160, 128, 96, 64, 32)}

    def cost(bm):
        rounds = tiles[bm] * columns / grid
        part = rounds - math.floor(rounds)
        return (math.floor(rounds) + (0.91 + 0.09 * part if part else 0)) * (4.24 + tiles[32] / tiles[bm])
    return min(tiles, key=cost)


MANY = np.random.default_rng(31).integers(0, 83, 300).tolist()


# N, and N - 8, whose last tile is cut; five K blocks, eleven with a short last one, seventeen
@pytest.mark.parametrize("sizes,N,Ks,want", [([17, 34, 17, 8] * 10, 1024, [2048, 2176], 32), ([350, 175] * 14, 1024, [640, 1296], 64),
                                             ([500, 1000, 1000], 2048, [640, 1296, 2176], 96), ([1158, 1158, 579], 2048, [640, 1296, 2176], 128),
                                             ([258, 517, 1034], 4096, [640, 1296, 2176], 160), (MANY, 512, [640, 2176], 64), ([150] * 280, 512, [640, 1296], 160)])
def test_every_height_that_the_kernel_chooses(sizes, N, Ks, want):
    """The automatic choice sends these to the fourth kernel, which chooses each of its five heights, and two of them over more
    groups than one index holds."""
    for n in (N, N - 8):
        assert torch.cuda.get_device_properties(0).multi_processor_count != 256 or chosen_height(sizes, n) == want
        for K in Ks:
            assert gg.auto_variant(len(sizes), sum(sizes), n, K) in (0, 3)
            check(problem(sizes, n, K, n + K), K, f"{len(sizes)} groups, N={n} K={K}")


def test_scales_that_are_nan_stay_in_their_rows():
    """A multiplying wave adds a row's last products in the next K block, also across tiles, and leaves out the steps that a tile
    does not have: nothing of one row may reach another."""
    sizes, N, K = [170, 5, 0, 330, 40, 96], 8192, 640
    A, SA, B, SB, off = problem(sizes, N, K, 3)
    bad = [0, 33, 169, 170, 200, 504, 545, 640]
    SA[bad] = float("nan")
    for v in (0, 3):
        for km in (False, True):
            C = gg.grouped_gemm(A, SA.t().contiguous() if km else SA, B, SB, off, variant=v, sa_kmajor=km)
            assert C.isnan().any(dim=1).nonzero().flatten().tolist() == bad, (v, km)


def test_against_the_oracle():
    sizes, N, K = [161, 0, 70, 3], 520, 1296
    dev = problem(sizes, N, K, 11)
    ref = orc.grouped_gemm(*(t.cpu().numpy() for t in dev), with_abs_sum=True)
    for v in (0, 3):
        assert_parity(bits_of(gg.grouped_gemm(*dev, variant=v)), ref, empirical=False, what=f"variant {v}")


def test_every_negative_variant_is_the_automatic_choice():
    sizes, N, K = [500, 1000, 1000], 2048, 640
    assert gg.auto_variant(len(sizes), sum(sizes), N, K) in (0, 3)
    dev = problem(sizes, N, K, 5)
    want = gg.grouped_gemm(*dev).view(torch.int16)
    for v in (-2, -27, -2 ** 31, -2 ** 31 + 25):
        assert torch.equal(gg.grouped_gemm(*dev, variant=v).view(torch.int16), want), v

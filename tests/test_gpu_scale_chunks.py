"""Row-major activation scales are fetched four K blocks at a time: numbers of K blocks around the multiples of four
(a last chunk of one, two, three blocks; fewer blocks than the ring has buffers), several tiles per workgroup so that
chunks run on from tile to tile.  The K-block-major order is fetched per K block and must give the same bits; one shape
is checked against the oracle as well."""
import numpy as np
import pytest
import torch

import paper_2508_16584_amd as gg
from oracle import gg_oracle as orc
from gg_testlib import assert_parity, bits_of

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


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


@pytest.mark.parametrize("K", [128, 256, 384, 512, 640, 1152, 1280, 1408, 1424])
def test_row_major_equals_kmajor_bitwise(K):
    sizes, N = [170, 0, 330, 40], 16384
    A, SA, B, SB, off = problem(sizes, N, K, K)
    SAk = SA.t().contiguous()
    want, ran = None, []
    for v in [-1] + list(range(gg.num_variants())):
        name = gg.variant_name(v) if v >= 0 else "auto"
        try:
            row = gg.grouped_gemm(A, SA, B, SB, off, variant=v)
            km = gg.grouped_gemm(A, SAk, B, SB, off, variant=v, sa_kmajor=True)
        except gg.GGError as e:
            assert e.status == 3 and v >= 0             # a variant that does not take this K
            continue
        ran.append(v)
        assert torch.equal(row.view(torch.int16), km.view(torch.int16)), name
        if "-rbk" not in name and "-k2" not in name:    # those add in an order of their own
            want = row if want is None else want
            assert torch.equal(row.view(torch.int16), want.view(torch.int16)), name
    # the tiles that take any K, the second kernel's from three K blocks on
    assert set(ran) >= {-1, 0, 2, 3, 5, 23, 24, 25} | ({12, 14, 15, 16} if K > 256 else set()) and (K % 256 or len(ran) == 1 + gg.num_variants() or K <= 256)


def test_row_major_against_the_oracle():
    sizes, N, K = [20, 3, 70], 512, 640
    dev = problem(sizes, N, K, 9)
    ref = orc.grouped_gemm(*(t.cpu().numpy() for t in dev), with_abs_sum=True)
    assert_parity(bits_of(gg.grouped_gemm(*dev)), ref, empirical=False, what="five K blocks")


@pytest.mark.parametrize("K", [4096, 4224, 4352, 4480, 4400])
def test_second_kernel_row_major_equals_kmajor_bitwise(K):
    """From K = 4096 on the second kernel fetches four K blocks of scales at a time too: last chunks of one to four
    blocks, even, odd and ragged numbers of K blocks, several tiles per workgroup.  A row's scales that are NaN stay in
    that row (what a chunk at the end of a row takes from the next one is not used, whatever it is)."""
    sizes, N = [700, 0, 300, 41], 8192
    A, SA, B, SB, off = problem(sizes, N, K, K)
    bad = [5, 17, 256, 700, 1040]
    SA[bad] = float("nan")
    SAk = SA.t().contiguous()
    want = gg.grouped_gemm(A, SAk, B, SB, off, variant=2, sa_kmajor=True)         # the first kernel, per K block
    any_k = [-1, 12, 14, 15, 16]                        # must run: the tiles with an instantiation for every K
    for v in [-1] + [u for u in range(gg.num_variants()) if gg.variant_name(u).endswith("-rb")]:
        try:
            row = gg.grouped_gemm(A, SA, B, SB, off, variant=v)
        except gg.GGError as e:
            assert e.status == 3 and v not in any_k     # whole K blocks, an even number of them, only
            continue
        assert torch.equal(row.view(torch.int16), want.view(torch.int16)) or \
            (torch.equal(row.isnan(), want.isnan()) and torch.equal(row.nan_to_num().view(torch.int16), want.nan_to_num().view(torch.int16))), v
        nan_rows = row.isnan().any(dim=1).nonzero().flatten().tolist()
        assert nan_rows == bad, v


@pytest.mark.parametrize("K", [2032, 2048, 2064, 2176, 2304, 2432])
def test_first_kernel_row_major_equals_kmajor_bitwise(K):
    """On such a problem every tile of the first kernel that can fetch four K blocks of scales at a time does so from K = 2048
    on: last chunks of one to four blocks, a ragged K, several tiles per workgroup; and NaN scales stay in their rows."""
    sizes, N = [170, 0, 330, 40], 16384
    A, SA, B, SB, off = problem(sizes, N, K, K)
    bad = [0, 169, 170, 333, 539]
    SA[bad] = float("nan")
    SAk = SA.t().contiguous()
    ran = []
    for v in range(gg.num_variants()):
        if "-rb" in gg.variant_name(v):
            continue
        try:
            row = gg.grouped_gemm(A, SA, B, SB, off, variant=v)
        except gg.GGError as e:
            assert e.status == 3                        # whole K blocks (an even number of them: split-K) only
            continue
        ran.append(v)
        km = gg.grouped_gemm(A, SAk, B, SB, off, variant=v, sa_kmajor=True)
        assert torch.equal(row.isnan(), km.isnan()) and torch.equal(row.nan_to_num().view(torch.int16), km.nan_to_num().view(torch.int16)), v
        assert row.isnan().any(dim=1).nonzero().flatten().tolist() == bad, v
    assert ran == [v for v in range(gg.num_variants()) if "-rb" not in gg.variant_name(v)
                   and (K % 128 == 0 or v in (0, 2, 3, 5, 23, 24, 25)) and (K % 256 == 0 or "-k2" not in gg.variant_name(v))]

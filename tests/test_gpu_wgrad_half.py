"""The weight gradient's narrow tiles halved where they can go wrong: numbers of token blocks around the ring of two buffers, groups
that begin and end inside blocks, empty ones, bytes of nobody's tokens that are NaN, tiles that don't come out even over the
workgroups, both outputs.  Against the oracle's hard bound, and bit for bit against the whole tiles, which the same tokens reach with the
rows of dY^T repeated (an output does not depend on how many others there are)."""
import numpy as np
import pytest
import torch

import paper_2508_16584_amd as gg
from oracle import gg_oracle as orc
from test_gpu_wgrad import assert_wgrad_parity, quantised_normal

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(off, M, N, K, seed):
    rng = np.random.default_rng(seed)
    XT, SX = quantised_normal(rng, K, M)
    DYT, SDY = quantised_normal(rng, N, M, std=0.02)
    G = len(off) - 1
    for lo, hi in ((0, off[0]), (off[-1], M)):             # nobody's tokens
        XT[:, lo:hi], DYT[:, lo:hi] = 0x7F, 0xFF
    assert gg.wgrad_route(G, M, N, K) == gg.wgrad_route(G, M, N, K, True) == {"half"}
    rep = 1
    while gg.wgrad_route(G, M, N * rep, K) or gg.wgrad_route(G, M, N * rep, K, True):
        rep += 1
    dev = lambda *xs: [torch.from_numpy(np.ascontiguousarray(x)).to(DEV) for x in xs]
    x, sx, y, sy, o = dev(XT, SX, DYT, SDY, np.asarray(off, np.int32))
    yn, syn = y.repeat(rep, 1), sy.repeat(1, rep)
    for bf16 in (False, True):
        got = gg.grouped_gemm_wgrad(x, sx, y, sy, o, out_bf16=bf16)
        whole = gg.grouped_gemm_wgrad(x, sx, yn, syn, o, out_bf16=bf16)
        bits = torch.int16 if bf16 else torch.int32
        assert torch.equal(got.view(bits), whole[:, -N:].contiguous().view(bits))
        if not bf16:
            ref = orc.grouped_gemm_wgrad(XT, SX, DYT, SDY, off, with_abs_sum=True)
            # the matrix instruction truncates the 8 products of a group to 2^-13 of the largest: 7 * 2^-13 of the absolute sum at most,
            # which a sum of seven tokens can come near (the others average it out)
            assert_wgrad_parity(got.cpu().numpy(), ref, 2.0 ** -10, f"{off}")
    for g in range(G):
        assert off[g] < off[g + 1] or (got[g] == 0).all()


@pytest.mark.parametrize("blocks", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("cut", [0, 16, 77])
def test_token_blocks_around_the_ring(blocks, cut):
    M = 128 * blocks + 16
    check([cut, 128 * blocks - (3 if cut else 0)], M, 1280, 2304, blocks + cut)


@pytest.mark.parametrize("off,M,N,K", [
    ([5, 5, 130, 300, 417, 417, 418, 500], 512, 640, 1280),      # fewer tiles than workgroups
    ([0] + [7 * g for g in range(1, 41)] + [280], 288, 384, 1024),       # more, and not a multiple of them
    ([0, 0, 0, 1, 1, 16, 16], 16, 1152, 1536),
    ([16, 555, 803, 804, 1190], 1200, 1408, 1280)])
def test_groups_that_cut_through_blocks(off, M, N, K):
    check(off, M, N, K, M)


def test_no_tokens_at_all():
    check([40, 40, 40], 48, 1024, 2048, 3)

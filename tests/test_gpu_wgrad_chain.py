"""The weight gradient's tiles of 64 x 64 (token blocks dealt to the waves) where they can go wrong: numbers of token blocks around what a
round of the four waves, one slot and both slots take, groups that begin and end inside blocks, empty ones, bytes of nobody's
tokens that are NaN, both outputs.  Against the oracle's bounds, and bit for bit against the narrow tiles, which the same tokens
reach with the rows of dY^T repeated (an output does not depend on how many others there are)."""
import numpy as np
import pytest
import torch

import paper_2508_16584_amd as gg
from oracle import gg_oracle as orc
from test_gpu_wgrad import assert_wgrad_parity, quantised_normal

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(off, M, N, K, seed, chain=True):
    rng = np.random.default_rng(seed)
    XT, SX = quantised_normal(rng, K, M)
    DYT, SDY = quantised_normal(rng, N, M, std=0.02)
    G = len(off) - 1
    for lo, hi in ((0, off[0]), (off[-1], M)):             # nobody's tokens
        XT[:, lo:hi], DYT[:, lo:hi] = 0x7F, 0xFF
    assert not chain or gg.wgrad_route(G, M, N, K) == gg.wgrad_route(G, M, N, K, True) == {"chain"}
    rep = 1
    while gg.wgrad_route(G, M, N * rep, K) or gg.wgrad_route(G, M, N * rep, K, True):
        rep *= 2
    dev = lambda *xs: [torch.from_numpy(np.ascontiguousarray(x)).to(DEV) for x in xs]
    x, sx, y, sy, o = dev(XT, SX, DYT, SDY, np.asarray(off, np.int32))
    yn, syn = dev(np.tile(DYT, (rep, 1)), np.tile(SDY, (1, rep)))
    for bf16 in (False, True):
        got = gg.grouped_gemm_wgrad(x, sx, y, sy, o, out_bf16=bf16)
        narrow = gg.grouped_gemm_wgrad(x, sx, yn, syn, o, out_bf16=bf16)
        bits = torch.int16 if bf16 else torch.int32
        assert torch.equal(got.view(bits), narrow[:, -N:].contiguous().view(bits))
        if not bf16:
            ref = orc.grouped_gemm_wgrad(XT, SX, DYT, SDY, off, with_abs_sum=True)
            assert_wgrad_parity(got.cpu().numpy(), ref, 2.0 ** -13, f"{off}")
    for g in range(G):
        assert off[g] < off[g + 1] or (got[g] == 0).all()


@pytest.mark.parametrize("blocks", [1, 2, 4, 5, 8, 9, 12, 13, 17])
@pytest.mark.parametrize("cut", [0, 16, 77])
def test_token_blocks_around_rounds_and_slots(blocks, cut):
    M = 128 * blocks + 16
    check([cut, 128 * blocks - (3 if cut else 0)], M, 128, 256, blocks + cut)


def test_groups_that_cut_through_blocks():
    check([5, 5, 256, 300, 901, 901, 902, 1270], 1280, 256, 512, 1, chain=False)
    check([16, 555, 1403, 1404, 1990], 2000, 384, 768, 2)


def test_no_tokens_at_all():
    check([40, 40, 40], 48, 128, 256, 3, chain=False)

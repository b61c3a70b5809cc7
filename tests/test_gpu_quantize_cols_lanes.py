"""The column quantiser with eight and with sixteen lanes per feature, on both sides of the line between them (three tiles of a token
block x 64 features per compute unit): every bf16 pattern, last blocks of 16, 112 and 128 tokens, tokens taken several times
and sources outside the input.  Against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from test_gpu_quantize_cols import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("more", [0, 1])                # sixteen lanes, eight
@pytest.mark.parametrize("last", [16, 112, 128])
@pytest.mark.parametrize("gather", [False, True])
def test_both_sides_of_the_line(more, last, gather):
    tiles = 3 * torch.cuda.get_device_properties(0).multi_processor_count
    K, blocks = 64 * 4, tiles // 4 + more
    rng = np.random.default_rng(8 * blocks + last + gather)
    T = M = 128 * (blocks - 1) + last
    src = None
    if gather:
        T = M // 3
        src = rng.integers(-2, T + 2, M)
    values = np.concatenate([np.arange(65536), rng.integers(0x3000, 0x4800, T * K)])[:T * K].astype(np.uint16)
    xb = rng.permutation(values).reshape(T, K)
    xb[:, :64] &= 0xBFFF                                 # features without infinities and NaNs
    check(xb, src)

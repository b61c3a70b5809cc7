"""The group of a tile is found by a ballot over tile counts summed up 64 groups at a time, groups past the first 256 by a
walk: numbers of groups around the multiples of 64 and beyond 256, most groups without rows, every variant."""
import numpy as np
import pytest
import torch

import paper_2508_16584_amd as gg
from oracle import gg_oracle as orc
from gg_testlib import assert_parity, bits_of

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("G", [1, 2, 63, 64, 65, 128, 129, 256, 257, 320, 700])
def test_every_variant_finds_every_group(G):
    rng = np.random.default_rng(G)
    N, K = 256, 384
    sizes = np.where(rng.random(G) < 0.3, rng.integers(1, 40, G), 0)
    sizes[rng.integers(0, G)] = 300
    sizes[-1] = 17
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    M = int(off[-1])
    A = rng.integers(0, 0x70, (M, K), dtype=np.uint8) | (rng.integers(0, 2, (M, K), dtype=np.uint8) << 7)
    B = rng.integers(0, 0x48, (G, N, K), dtype=np.uint8) | (rng.integers(0, 2, (G, N, K), dtype=np.uint8) << 7)
    SA = rng.uniform(0.5, 2.0, (M, K // 128)).astype(np.float32)
    SB = rng.uniform(0.5, 2.0, (G, N // 128, K // 128)).astype(np.float32)
    ref = orc.grouped_gemm(A, SA, B, SB, off, with_abs_sum=True)
    dev = tuple(torch.from_numpy(x).to(DEV) for x in (A, SA, B, SB, off))
    want, ran = None, []
    for v in [-1] + list(range(gg.num_variants())):
        try:
            got = bits_of(gg.grouped_gemm(*dev, variant=v))
        except gg.GGError as e:
            assert e.status == 3 and v >= 0             # a variant that does not take this K: three K blocks
            continue
        ran.append(v)
        assert_parity(got, ref, empirical=False, what=f"G={G} variant {v}")
        if v < 0 or not gg.variant_name(v).endswith("-rbk"):      # (adds in an order of its own)
            want = got if want is None else want
            assert np.array_equal(got, want), f"variant {v} differs"
    # all but split-K (an even number of K blocks) and those of the second kernel that have no instantiation for an odd one
    assert ran == [-1] + [v for v in range(gg.num_variants()) if "-k2" not in gg.variant_name(v)
                          and ("-rb" not in gg.variant_name(v) or gg.variant_name(v)[:3] in ("256", "224", "192", "128") and gg.variant_name(v).endswith("-rb"))]

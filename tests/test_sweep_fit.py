"""sweep.py's fit of the small tiles: it has the form of the library's estimates, so it finds the constants that made the times."""
import math
import os
import re

import numpy as np
import pytest

import sweep

SOURCE = os.path.join(os.path.dirname(os.path.abspath(sweep.__file__)), "paper_2508_16584_amd", "csrc", "gg_fp8.hip")


def problems(seed, n=600):
    rng = np.random.default_rng(seed)
    draw = lambda lo, hi, step=1: max(lo, int(lo * (hi / lo) ** rng.random() / step) * step)
    return [(draw(1, 256), draw(1, 32768), draw(256, 8192, 128), draw(256, 8192, 128)) for _ in range(n)]


def chain_us(G, M, N, K, BM, BN, per_cu, waves, latency, work, extra, start):          # estimate_chain_us
    groups = G * (1 - math.exp(-M / G))
    tiles, steps = max(groups, M / BM + 0.5 * groups) * -(-N // BN), -(-K // (128 * waves)) + extra
    a, b, c = max(tiles / (256 * per_cu), 1) * steps * latency, tiles * steps * work / 256, (groups * N * K + M * (K + 2 * N)) / 6.8e6
    return start + (a ** 4 + b ** 4 + c ** 4) ** 0.25


@pytest.mark.parametrize("v", [26, 27, 28])
def test_the_fifth_kernels_constants_are_found(v):
    BM, BN, _, per_cu, waves = tile = sweep.SMALL_TILES[v]
    source = open(SOURCE).read()
    times = re.search(r"kChainTimes\[\] = \{(.*)\};", source).group(1)
    want = [float(x) for x in re.search(r"\{%d, ([^}]*)\}" % v, times).group(1).split(",")]      # latency, work, extra, start, waves
    assert want.pop() == waves
    rows = [dict(G=G, M=M, N=N, K=K, us={v: chain_us(G, M, N, K, BM, BN, per_cu, waves, *want)}) for G, M, N, K in problems(v)]
    got, error, half = sweep.fit_tile(rows, v, tile, False)
    assert half == 300 and error < 0.01 and np.allclose(got, want, rtol=0.05), (got, want)

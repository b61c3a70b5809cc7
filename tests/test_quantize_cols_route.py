"""How the column quantiser runs (gg_fp8_quantize_cols_route)."""
import pytest
import torch

import paper_2508_16584_amd as gg


def test_strips_only_where_rows_of_the_output_are_whole_lines():
    """A row that starts inside a line, by the tensor's address or by the row before it, shares lines with its neighbour."""
    T, M, K = 8192, 16384, 8192
    buf = torch.empty(512, dtype=torch.uint8)
    buf = buf[-buf.data_ptr() % 128:]
    assert "strips" in gg.quantize_cols_route(T, M, K, buf)
    for first in (16, 64, 112):
        assert not gg.quantize_cols_route(T, M, K, buf[first:])
    assert not gg.quantize_cols_route(T, M - 16, K, buf)


def test_strips_only_where_the_gather_takes_tokens_a_few_times():
    """Not where next to every token is read once, in the order that a token's neighbours come in (a routing that keeps all of them
    but a few), and not where the input is so much smaller that it stays in the caches whatever the order is."""
    M = 16384
    for K in (6144, 7168, 8192):
        for T in (8192, 4096):
            assert "strips" in gg.quantize_cols_route(T, M, K)
        for T in (M, M - 1, M - 16, M - 1024, M // 8, M // 64, 1):
            assert "strips" not in gg.quantize_cols_route(T, M, K), T


def test_what_the_call_refuses_has_no_route():
    for T, M, K in [(-1, 128, 128), (16, 129, 128), (16, 128, 96), (16, 128, 1 << 23)]:
        with pytest.raises(ValueError):
            gg.quantize_cols_route(T, M, K)

"""How the weight-gradient call runs (gg_fp8_wgrad_route), as far as it must not depend on sizes that were measured."""
import pytest
import torch

import paper_2508_16584_amd as gg


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


def test_what_the_call_refuses_has_no_route():
    for G, M, N, K in [(-1, 16, 256, 256), (4, 17, 256, 256), (4, 16, 200, 256), (4, 16, 256, 128), (4, 1 << 24, 256, 256), (4, 16, 256, 1 << 21)]:
        with pytest.raises(ValueError):
            gg.wgrad_route(G, M, N, K)
    assert gg.wgrad_route(0, 16, 256, 256) == set()

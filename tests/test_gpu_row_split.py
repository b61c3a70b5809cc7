"""How the row kernels (quantiser, activation + quantiser) split their work: several short rows per workgroup, a row in
several pieces, runs of rows per XCD with K-block-major scales, streaming stores.  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import paper_2508_16584_amd as gg
from oracle import gg_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def rows_of(T, K, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return (torch.randn((T, K), generator=gen, device=DEV) * torch.randn((T, 1), generator=gen, device=DEV).exp()).to(torch.bfloat16)


def bits(t):
    return t.cpu().view(torch.int16).numpy().view(np.uint16)


# K / 128 = 1, 3 (21 rows per pass with a slot left over), 33 (more than half a pass), 63, 64 (a pass to the block), 65 and
# 129 (two and three pieces); row counts around the runs of 8 x 8 and 8 x 32 rows
@pytest.mark.parametrize("M,K", [(1, 128), (1300, 128), (700, 384), (65, 4224), (63, 8064), (257, 8192), (64, 8320), (9, 16512),
                                 (2049, 8192)])
@pytest.mark.parametrize("km", [False, True])
def test_quantiser_split(M, K, km):
    T = M // 2 + 1
    X = rows_of(T, K, M + K)
    src = torch.from_numpy(np.random.default_rng(M).integers(-1, T + 1, M).astype(np.int32)).to(DEV)
    A, SA = gg.quantize_rows(X, src, sa_kmajor=km, A=torch.full((M, K), 0xA5, dtype=torch.uint8, device=DEV),
                             SA=torch.full((K // 128, M) if km else (M, K // 128), -7.0, device=DEV))
    torch.cuda.synchronize()
    A_ref, SA_ref = orc.quantize_rows(bits(X), src.cpu().numpy(), M)
    assert np.array_equal(A.cpu().numpy(), A_ref)
    assert np.array_equal((SA.t() if km else SA).contiguous().cpu().numpy().view(np.uint32), SA_ref.view(np.uint32))


# I / 128 = 1, 11 (two rows and ten slots left), 31, 32, 33
@pytest.mark.parametrize("M,inter", [(1, 128), (1100, 128), (601, 1408), (40, 3968), (257, 4096), (33, 4224)])
@pytest.mark.parametrize("km", [False, True])
def test_activation_split(M, inter, km):
    H = rows_of(M, 2 * inter, M + inter)
    A, SA, act = gg.swiglu_quantize_rows(H, want_act=True, sa_kmajor=km)
    torch.cuda.synchronize()
    A_ref, SA_ref = orc.quantize_rows(bits(act), None, M)         # bytes and scales follow from the activations
    assert np.array_equal(A.cpu().numpy(), A_ref)
    assert np.array_equal((SA.t() if km else SA).contiguous().cpu().numpy().view(np.uint32), SA_ref.view(np.uint32))
    g, u = H[:, :inter].double(), H[:, inter:].double()
    ref = g * torch.sigmoid(g) * u
    # half a bf16 ulp (2^-9 of the value) and the fp32 evaluation, far below another half
    assert bool(((act.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-30).all())


# The tests above have up to 32 blocks per compute unit but for three of them: sixteen lanes per block.  The same splits with
# eight lanes, just above 8192 blocks, and both sides of the line.
@pytest.mark.parametrize("M,K", [(8192, 128), (8193, 128), (2731, 384), (249, 4224), (131, 8064), (127, 8320), (65, 16512)])
@pytest.mark.parametrize("km", [False, True])
def test_quantiser_split_above_the_line(M, K, km):
    test_quantiser_split(M, K, km)


@pytest.mark.parametrize("M,inter", [(8192, 128), (8193, 128), (745, 1408), (265, 3968), (249, 4224)])
@pytest.mark.parametrize("km", [False, True])
def test_activation_split_above_the_line(M, inter, km):
    test_activation_split(M, inter, km)


@pytest.mark.parametrize("K", [256, 16640])                       # 2 and 130 blocks per row
def test_both_lane_counts_agree(K):
    """Infinities, NaNs, zeros, denormals and the largest values: the same rows in a call of few blocks and in one of many."""
    rows = 8192 // (K // 128) + 1
    special = torch.tensor([0x0000, 0x8000, 0x0001, 0x8001, 0x7F7F, 0xFF7F, 0x7F80, 0xFF80, 0x7FC0, 0xFFC1, 0x7F81, 0x0080], device=DEV).to(torch.int32)
    X = rows_of(rows, K, K).view(torch.int16)
    mask = torch.rand(X.shape, device=DEV) < 0.01
    X = torch.where(mask, special[torch.randint(0, 12, X.shape, device=DEV)].to(torch.int16), X).view(torch.bfloat16)
    A, SA = gg.quantize_rows(X)
    B, SB = gg.quantize_rows(X[-37:].contiguous())
    assert torch.equal(A[-37:], B) and torch.equal(SA[-37:].view(torch.int32), SB.view(torch.int32))
    H = X.view(-1, K)
    A, SA, act = gg.swiglu_quantize_rows(torch.cat([H, H]), want_act=True)
    B, SB, act_b = gg.swiglu_quantize_rows(H[-37:].contiguous(), want_act=True)
    assert torch.equal(A[-37:], B) and torch.equal(SA[-37:].view(torch.int32), SB.view(torch.int32))
    assert torch.equal(act[-37:].view(torch.int16), act_b.view(torch.int16))


def test_streaming_stores_equal_the_others():
    """128 MB of bytes and more: the instantiations with streaming stores (rows read again, activations) and loads, against the
    others on some of the same rows."""
    X = rows_of(14400, 7168, 5)
    A, SA = gg.quantize_rows(X)
    B, SB = gg.quantize_rows(X[7000:7500])
    assert torch.equal(A[7000:7500], B) and torch.equal(SA[7000:7500], SB)
    src = torch.randint(0, 500, (18800,), device=DEV, dtype=torch.int32)        # rows read again
    A, SA = gg.quantize_rows(X[7000:7500], src)
    assert torch.equal(A, B[src.long()]) and torch.equal(SA, SB[src.long()])
    H = X.view(-1, 256)
    H = torch.cat([H, H, H])
    A2, SA2, _ = gg.swiglu_quantize_rows(H)
    B2, SB2, _ = gg.swiglu_quantize_rows(H[-700:])
    assert torch.equal(A2[-700:], B2) and torch.equal(SA2[-700:], SB2)

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


def test_streaming_stores_equal_the_others():
    """More than 96 MB of bytes: the instantiations with streaming stores, against the others on some of the same rows."""
    X = rows_of(14400, 7168, 5)
    A, SA = gg.quantize_rows(X)
    B, SB = gg.quantize_rows(X[7000:7500])
    assert torch.equal(A[7000:7500], B) and torch.equal(SA[7000:7500], SB)
    src = torch.randint(0, 500, (15000,), device=DEV, dtype=torch.int32)        # rows read again
    A, SA = gg.quantize_rows(X[7000:7500], src)
    assert torch.equal(A, B[src.long()]) and torch.equal(SA, SB[src.long()])
    H = X.view(-1, 256)
    H = torch.cat([H, H])
    A2, SA2, _ = gg.swiglu_quantize_rows(H)
    B2, SB2, _ = gg.swiglu_quantize_rows(H[-700:])
    assert torch.equal(A2[-700:], B2) and torch.equal(SA2[-700:], SB2)

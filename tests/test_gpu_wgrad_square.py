"""gg_fp8_grouped_gemm_wgrad on launches large enough for its tiles of 256 x 256.

Every intermediate is exact (integers up to 4, scales 1/2, 1 and 2, at most 2100 tokens per group: sums below 2^24 in units of
1/4), so the fp32 result must equal the product in float64, and the bfloat16 one its rounding.  One group's tokens are NaN in
both operands: its neighbours fetch some of them in their first and last 16 tokens and must not show them.
"""
import pytest
import torch

import paper_2508_16584_amd as gg

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LENGTHS = [1, 0, 16, 15, 127, 128, 129, 400, 512, 513, 0, 900, 3]


def check_exact(sizes, nan, N, K, out_bf16, seed):
    """Groups of these sizes, those of group `nan` NaN; returns how the call ran."""
    G = len(sizes)
    off = torch.tensor([0] + sizes).cumsum(0) + 5
    M = -(-int(off[-1]) // 16) * 16
    MB = -(-M // 128)
    gen = torch.Generator(device=DEV).manual_seed(seed)

    def operand(rows):
        v = torch.randint(-4, 5, (rows, M), generator=gen, device=DEV).float()
        s = 2.0 ** torch.randint(-1, 2, (MB, rows), generator=gen, device=DEV).float()
        exact = v * s.t().repeat_interleave(128, dim=1)[:, :M]
        q = v.to(torch.float8_e4m3fn).view(torch.uint8)
        q[:, off[nan]:off[nan + 1]] = 0x7F
        q[:, :5] = 0xFF                          # nobody's tokens
        return q, s, exact

    XT, SX, X = operand(K)
    DYT, SDY, DY = operand(N)
    got = gg.grouped_gemm_wgrad(XT, SX, DYT, SDY, off.int().to(DEV), out_bf16=out_bf16)
    for g in range(G):
        if g == nan:
            assert torch.isnan(got[g]).all()
            continue
        want = (DY[:, off[g]:off[g + 1]].double() @ X[:, off[g]:off[g + 1]].double().t().contiguous()).float()
        assert torch.equal(got[g], want.bfloat16() if out_bf16 else want), (g, sizes[g])
    return gg.wgrad_route(G, M, N, K, out_bf16, SX, SDY)


# runs of tiles dealt by cost: whole ones, a partial one per group; listed in order: more than 64 groups, few token blocks per group
@pytest.mark.parametrize("N,K,G,mean,way", [(5120, 4096, 8, 1100, {"square", "dealt"}), (4608, 4352, 9, 900, {"square", "dealt"}),
                                            (2560, 2304, 70, 270, {"square"}), (3840, 3072, 41, 200, {"square"})])
@pytest.mark.parametrize("out_bf16", [False, True])
def test_exact_over_lengths(N, K, G, mean, way, out_bf16):
    gen = torch.Generator().manual_seed(N + G)
    sizes = [LENGTHS[i] for i in torch.randint(0, len(LENGTHS), (G,), generator=gen).tolist()]
    nan, i = G // 2, 0
    sizes[nan] = 35
    while sum(sizes) < mean * G:                 # groups of many blocks, until the launch is one for these tiles
        if i != nan:
            sizes[i] = 2100 - i
        i += 1
    assert way <= check_exact(sizes, nan, N, K, out_bf16, seed=G)


# The operands brought in ahead beside tiles of no and of one token block: their fetches are counted with the stores.  Dealt out,
# and (more than 64 groups) in order.
@pytest.mark.parametrize("G,long,way", [(24, 2400, {"square", "ahead", "dealt"}), (72, 900, {"square", "ahead"})])
@pytest.mark.parametrize("out_bf16", [False, True])
def test_operands_ahead_of_short_tiles(G, long, way, out_bf16):
    sizes = [(0, 0, long, 1, 128, 0, long - 77, 0, 16, 35)[g % 10] for g in range(G)]
    sizes[0] += 1500
    assert check_exact(sizes, 19, 3840, 4096, out_bf16, seed=G) == way


# Operands of 80 MB and more are brought into the last-level cache first: token counts that are and are not whole pieces of
# 1024, rows that do and do not divide over the waves
@pytest.mark.parametrize("M,N,K,G", [(8192, 4096, 7168, 8), (9008, 6144, 3328, 10), (15376, 2560, 5120, 28),
                                     (16384, 7168, 2048, 32)])
def test_large_operands(M, N, K, G):
    assert gg.wgrad_route(G, M, N, K) == {"square", "ahead", "dealt"}
    gen = torch.Generator(device=DEV).manual_seed(M)
    XT = torch.randint(0, 2, (K, M), generator=gen, device=DEV, dtype=torch.uint8) * 0x38          # 0 and 1
    DYT = torch.randint(0, 2, (N, M), generator=gen, device=DEV, dtype=torch.uint8) * 0x40         # 0 and 2
    one = lambda rows: torch.ones((-(-M // 128), rows), device=DEV)
    off = torch.linspace(0, M, G + 1).int()
    off[1] -= 77
    got = gg.grouped_gemm_wgrad(XT, one(K), DYT, one(N), off.to(DEV))
    X, DY = (XT != 0).float(), (DYT != 0).float() * 2          # products of small integers: exact in float32
    for g in range(G):
        assert torch.equal(got[g], DY[:, off[g]:off[g + 1]] @ X[:, off[g]:off[g + 1]].t().contiguous()), g


# Offsets past the ends and out of order, as the header promises: clamped, a group that ends before it starts has no tokens
@pytest.mark.parametrize("N,K,way", [(5120, 4096, {"square", "dealt"}), (8192, 2048, {"square"})])
def test_bad_offsets_are_clamped(N, K, way):
    bad = [-50, 1000, 900, 3000, 3001, 20000, 5000, 8000, 8990, 30000, 12000]
    M, G = 12000, len(bad) - 1
    if "dealt" not in way:
        bad, G = bad + [M] * 20, G + 20                # whole rounds per group: nothing to deal
    assert way <= gg.wgrad_route(G, M, N, K)
    gen = torch.Generator(device=DEV).manual_seed(N)
    XT = torch.randint(0, 2, (K, M), generator=gen, device=DEV, dtype=torch.uint8) * 0x38          # 0 and 1
    DYT = torch.randint(0, 2, (N, M), generator=gen, device=DEV, dtype=torch.uint8) * 0x40         # 0 and 2
    one = lambda rows: torch.ones((-(-M // 128), rows), device=DEV)
    got = gg.grouped_gemm_wgrad(XT, one(K), DYT, one(N), torch.tensor(bad, dtype=torch.int32, device=DEV))
    X, DY = (XT != 0).float(), (DYT != 0).float() * 2
    for g in range(G):
        lo = min(max(bad[g], 0), M)
        hi = min(max(bad[g + 1], lo), M)
        assert torch.equal(got[g], DY[:, lo:hi] @ X[:, lo:hi].t().contiguous()), g


def test_scales_that_start_between_two_16_byte_pieces():
    """They stay with the narrow tiles, which fetch four bytes per lane; the result is the same."""
    G, M, N, K = 8, 8192, 8192, 7936
    gen = torch.Generator(device=DEV).manual_seed(1)
    XT = torch.randint(0, 120, (K, M), generator=gen, device=DEV, dtype=torch.uint8)
    DYT = torch.randint(0, 120, (N, M), generator=gen, device=DEV, dtype=torch.uint8)
    off = torch.tensor([0, 1000, 1000, 3000, 4003, 5500, 5501, 7900, M], dtype=torch.int32, device=DEV)

    def scales(rows, first):
        s = torch.rand((M // 128, rows), generator=torch.Generator(device=DEV).manual_seed(2), device=DEV)
        flat = torch.empty(s.numel() + first, device=DEV)
        flat[first:] = s.view(-1)
        return flat[first:].view(M // 128, rows)

    assert "square" in gg.wgrad_route(G, M, N, K, True, scales(K, 0), scales(N, 0))
    want = gg.grouped_gemm_wgrad(XT, scales(K, 0), DYT, scales(N, 0), off, out_bf16=True)
    for a, b in ((1, 0), (0, 3)):
        assert not gg.wgrad_route(G, M, N, K, True, scales(K, a), scales(N, b))
        assert torch.equal(gg.grouped_gemm_wgrad(XT, scales(K, a), DYT, scales(N, b), off, out_bf16=True).view(torch.int16), want.view(torch.int16))

"""Seeded random shapes through every entry point that takes them: the padding-free GEMM against the oracle, element
by element, and the identities that tie the other paths to it (K-block-major scales, pad path, fused activation
epilogue: all bit for bit).  The draws favour the edges: empty groups, groups of one row, group sizes next to tile
heights, N and K that are and are not multiples of 128 and 256."""
import numpy as np
import pytest
import torch

import paper_2508_16584_amd as gg
from oracle import gg_oracle as orc
from gg_testlib import assert_parity, bits_of

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def draw(seed, long=False):
    rng = np.random.default_rng(seed)
    G = int(rng.integers(1, 7))
    edge = np.array([0, 1, 15, 16, 17, 127, 128, 129, 159, 160, 161, 191, 192, 193, 223, 224, 225, 255, 256, 257, 400])
    sizes = np.where(rng.random(G) < 0.6, rng.choice(edge, G), rng.integers(0, 500, G))
    N = int(rng.choice([8, 64, 128, 136, 256, 384, 512, 520, 768, 1024]))
    K = int(rng.choice([1280, 2048, 2064, 2176, 4096, 4224, 4240, 4352, 4480] if long else [16, 128, 144, 256, 512, 768, 1024, 1040, 1536, 2048]))
    return rng, sizes, N, K


def problem(seed, long=False):
    rng, sizes, N, K = draw(seed, long)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    M, G = int(off[-1]), len(sizes)
    KB, NB = -(-K // 128), -(-N // 128)
    A = rng.integers(0, 256, (max(M, 1), K), dtype=np.uint8)[:M]
    B = rng.integers(0, 256, (G, N, K), dtype=np.uint8)
    A[(A & 0x7F) == 0x7F] = 0x35
    B[(B & 0x7F) == 0x7F] = 0x35
    A[(A & 0x78) > 0x58] &= 0xBF                 # moderate magnitudes: finite bf16 results with scales up to 4
    B[(B & 0x78) > 0x50] &= 0xBF
    SA = rng.uniform(0.25, 4.0, (M, KB)).astype(np.float32)
    SB = rng.uniform(0.25, 4.0, (G, NB, KB)).astype(np.float32)
    return sizes, (A, SA, B, SB, off)


@pytest.mark.parametrize("seed", range(7000, 7016))
def test_random_shape_all_paths(seed):
    sizes, (A, SA, B, SB, off) = problem(seed)
    (M, K), (G, N, _) = A.shape, B.shape
    dA, dSA, dB, dSB, doff = (torch.from_numpy(np.ascontiguousarray(x)).to(DEV) for x in (A, SA, B, SB, off))
    what = f"seed {seed}: sizes {sizes.tolist()} N={N} K={K}"
    C = gg.grouped_gemm(dA, dSA, dB, dSB, doff, C=torch.zeros((M, N), dtype=torch.bfloat16, device=DEV))
    torch.cuda.synchronize()
    if M > 0:
        ref = orc.grouped_gemm(A, SA, B, SB, off, with_abs_sum=True)
        assert_parity(bits_of(C), ref, empirical=False, what=what)
    # K-block-major scales
    SAk = dSA.t().contiguous()
    Ck = gg.grouped_gemm(dA, SAk, dB, dSB, doff, C=torch.zeros((M, N), dtype=torch.bfloat16, device=DEV), sa_kmajor=True)
    # pad path, both orders
    outs = [Ck]
    for km in (False, True):
        A_pad, SA_pad, poff = gg.pad(dA, SAk if km else dSA, doff, sa_kmajor=km)
        C_pad = gg.grouped_gemm_padded(A_pad, SA_pad, dB, dSB, poff, sa_kmajor=km)
        outs.append(gg.unpad(C_pad, doff, poff, M, C=torch.zeros((M, N), dtype=torch.bfloat16, device=DEV)))
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        assert torch.equal(o.view(torch.int16), C.view(torch.int16)), f"{what}: path {i} differs from the padding-free result"
    # the activation epilogue, where the shape allows it (and the plain GEMM adds the K blocks in the same order)
    if N % 256 == 0 and K % 128 == 0 and K > 256 and K % 8192 != 4096:
        A2r, S2r, actr = gg.swiglu_quantize_rows(C, want_act=True)
        for km in (False, True):
            A2, S2, act = gg.grouped_gemm_swiglu(dA, SAk if km else dSA, dB, dSB, doff, want_act=True, sa_kmajor=km,
                                                 A2=torch.zeros((M, N // 2), dtype=torch.uint8, device=DEV),
                                                 SA2=torch.zeros((N // 256, M) if km else (M, N // 256), dtype=torch.float32, device=DEV),
                                                 act_out=torch.zeros((M, N // 2), dtype=torch.bfloat16, device=DEV))
            torch.cuda.synchronize()
            # zero-filled outputs: rows of empty problems stay zero on both sides
            if M > 0:
                assert torch.equal(A2, A2r), f"{what}: fused bytes"
                assert torch.equal(act.view(torch.int16), actr.view(torch.int16)), f"{what}: fused activations"
                assert torch.equal((S2.t().contiguous() if km else S2).view(torch.int32), S2r.view(torch.int32)), f"{what}: fused scales"


# variants with an instantiation for partial tiles and a short last K block (the second kernel: for an odd number of K blocks)
RAGGED_TILES = ("160x256/2x4w/3s", "128x128/2x4w/4s", "128x256/2x4w/3s", "32x256/1x8w/4s", "256x256/1x8w/3s-rb", "192x256/1x8w/3s-rb",
                "224x256/1x8w/3s-rb", "128x256/1x8w/3s-rb", "32x64/2x2w/4s", "32x128/1x4w/3s", "64x128/2x2w/3s")


def takes(name, N, K):
    """Whether the tile takes this N and K: the rule of include/gg_fp8.h."""
    BN, second, split = int(name.split("/")[0].split("x")[1]), "-rb" in name, name.endswith("-k2")
    ragged = N % BN != 0 or K % 128 != 0 or (second and -(-K // 128) % 2 == 1)
    return not (ragged and name not in RAGGED_TILES) and not (second and K <= 256) and not (split and (K % 256 != 0 or N % BN != 0))


@pytest.mark.parametrize("seed", list(range(7000, 7016)) + list(range(7100, 7110)))
def test_random_shape_every_tile(seed):
    """The automatic choice takes small tiles on problems of this size: every tile that the shape allows by name, in both scale
    orders, and the activation epilogue of every tile that has one.  The same bits as the automatic result; the two kinds
    that add the K blocks in an order of their own against the oracle.  Seeds from 7100 on draw long K loops, where row-major
    scales are fetched four K blocks at a time."""
    sizes, host = problem(seed, long=seed >= 7100)
    (M, K), (G, N, _) = host[0].shape, host[2].shape
    if M == 0:
        pytest.skip("no rows")
    dA, dSA, dB, dSB, doff = (torch.from_numpy(np.ascontiguousarray(x)).to(DEV) for x in host)
    orders = {False: dSA, True: dSA.t().contiguous()}
    what = f"seed {seed}: sizes {sizes.tolist()} N={N} K={K}"
    C = gg.grouped_gemm(dA, dSA, dB, dSB, doff)
    ref = orc.grouped_gemm(*host, with_abs_sum=True)
    assert_parity(bits_of(C), ref, empirical=False, what=what)
    for v in range(gg.num_variants()):
        name = gg.variant_name(v)
        for km, scales in orders.items():
            out = torch.zeros((M, N), dtype=torch.bfloat16, device=DEV)
            if not takes(name, N, K):
                with pytest.raises(gg.GGError) as e:
                    gg.grouped_gemm(dA, scales, dB, dSB, doff, C=out, variant=v, sa_kmajor=km)
                assert e.value.status == 3, name
                continue
            gg.grouped_gemm(dA, scales, dB, dSB, doff, C=out, variant=v, sa_kmajor=km)
            if name.endswith("-rbk") or name.endswith("-k2"):
                assert_parity(bits_of(out), ref, empirical=False, what=f"{what} {name}")
            else:
                assert torch.equal(out.view(torch.int16), C.view(torch.int16)), f"{what}: {name}, K-block-major {km}"
    if N % 256 == 0 and K % 128 == 0 and K > 256 and K % 8192 != 4096:
        A2r, S2r, actr = gg.swiglu_quantize_rows(C, want_act=True)
        for name in ("192x256/1x8w/3s-rb", "224x256/1x8w/3s-rb", "256x256/1x8w/3s-rb", "32x128/1x4w/3s", "64x128/2x2w/3s"):
            v = next(v for v in range(gg.num_variants()) if gg.variant_name(v) == name)
            if K % 256 != 0 and name[:3] in ("224", "256"):
                continue
            for km, scales in orders.items():
                A2, S2, act = gg.grouped_gemm_swiglu(dA, scales, dB, dSB, doff, want_act=True, sa_kmajor=km, variant=v)
                assert torch.equal(A2, A2r) and torch.equal(act.view(torch.int16), actr.view(torch.int16)), f"{what}: fused {name}"
                assert torch.equal((S2.t().contiguous() if km else S2).view(torch.int32), S2r.view(torch.int32)), f"{what}: fused {name}"

"""gg_fp8_swiglu_route: which fused calls run as two launches, and that the two give the bytes of the one."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2508_16584_amd as gg
from paper_2508_16584_amd import binding

DEV = "cuda:0"


def route(G, M, I, K, flags=0):
    return gg.load_library().gg_fp8_swiglu_route(G, M, I, K, flags)


def test_sizes():
    assert route(37, 1, 640, 7808) == 1 and route(8, 64, 512, 2048) == 1            # few tiles of 256 weight rows
    assert route(8, 8192, 2048, 7168) == 0                                         # 64 MB of intermediate, and as fast in one
    assert route(1, 1 << 20, 2048, 7168) == 0                                      # 8 GB
    assert route(4, 3, 256, 4096) == 0 and route(4, 3, 256, 4096 + 8192) == 0      # K loops that begin elsewhere in the plain GEMM
    assert route(0, 0, 256, 512) == 0 and route(3, 0, 256, 512) == 0
    lib = gg.load_library()                                                        # what the fused call refuses
    for G, M, I, K, flags in [(4, 8, 64, 512, 0), (4, 8, 256, 256, 0), (4, 8, 256, 400, 0), (4, 8, 256, 512, 1), (-1, 8, 256, 512, 0), (4, 8, 1 << 20, 1 << 20, 0)]:
        null = ctypes.c_void_p()
        assert route(G, M, I, K, flags) == -lib.gg_fp8_grouped_gemm_swiglu(*[null] * 8, G, M, I, K, null, -1, flags) < 0


@pytest.mark.parametrize("km", [False, True])
@pytest.mark.parametrize("want_act", [False, True])
@pytest.mark.parametrize("room,launches", [("outputs", 1), ("outputs and most of the intermediate", 1), ("outputs and intermediate", 2)])
def test_outputs_are_allocated_before_the_intermediate(room, launches, want_act, km, monkeypatch):
    """The binding's Python form on CPU tensors, with an allocator of limited room and a library that launches nothing."""
    G, M, I, K = 4, 64, 256, 512
    assert route(G, M, I, K, 2 if km else 0) == 1
    made = []

    class Library:
        gg_fp8_swiglu_route = gg.load_library().gg_fp8_swiglu_route

        def __getattr__(self, name):
            return (lambda *args: 0) if name.startswith("gg_fp8_workspace") else lambda *args: made.append(name) or 0

    cpu = [torch.zeros(M, K, dtype=torch.uint8), torch.zeros((K // 128, M) if km else (M, K // 128)), torch.zeros(G, 2 * I, K, dtype=torch.uint8),
           torch.zeros(G, 2 * I // 128, K // 128), torch.zeros(G + 1, dtype=torch.int32)]
    outputs, H = M * I + 4 * M * I // 128 + (2 * M * I if want_act else 0), 4 * M * I
    left = [{"outputs": outputs, "outputs and most of the intermediate": outputs + H - 1, "outputs and intermediate": outputs + H}[room]]
    empty = torch.empty

    def limited(*args, **kw):
        t = empty(*args, **kw)
        if t.nbytes > left[0]:
            raise torch.OutOfMemoryError("no room")
        left[0] -= t.nbytes
        return t

    monkeypatch.setattr(binding, "_calls", None)
    monkeypatch.setattr(binding, "_want", lambda *args: None)
    monkeypatch.setattr(binding, "_stream", lambda stream: None)
    monkeypatch.setattr(binding, "load_library", Library)
    monkeypatch.setattr(torch, "empty", limited)
    A2, SA2, act = gg.grouped_gemm_swiglu(*cpu, want_act=want_act, sa_kmajor=km)
    assert A2.shape == (M, I) and SA2.shape == ((I // 128, M) if km else (M, I // 128)) and (act is not None) == want_act
    assert len(made) == launches and ("swiglu" in made[0]) == (launches == 1)


def problem(sizes, I, K, seed):
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    M, G = int(off[-1]), len(sizes)
    A = rng.integers(0, 0x50, (M, K), dtype=np.uint8) | (rng.integers(0, 2, (M, K), dtype=np.uint8) << 7)
    B = rng.integers(0, 0x30, (G, 2 * I, K), dtype=np.uint8) | (rng.integers(0, 2, (G, 2 * I, K), dtype=np.uint8) << 7)
    SA = rng.uniform(0.5, 2.0, (M, K // 128)).astype(np.float32)
    SB = rng.uniform(0.5, 2.0, (G, 2 * I // 128, K // 128)).astype(np.float32)
    return [torch.from_numpy(x).to(DEV) for x in (A, SA, B, SB, off)]


@pytest.mark.gpu
@pytest.mark.parametrize("sizes,I,K", [([1], 128, 384), ([0, 3, 17, 1], 640, 1152), ([5, 40], 256, 2176), ([30] * 8, 384, 512)])
@pytest.mark.parametrize("km", [False, True])
@pytest.mark.parametrize("native", [True, False])
def test_two_launches_give_the_bytes_of_the_fused_kernel(sizes, I, K, km, native, monkeypatch):
    dev = problem(sizes, I, K, K)
    if km:
        dev[1] = dev[1].t().contiguous()
    one = next(v for v in range(gg.num_variants()) if gg.variant_name(v) == "32x128/1x4w/3s")
    want = gg.grouped_gemm_swiglu(*dev, want_act=True, sa_kmajor=km, variant=one)
    if not native:
        monkeypatch.setattr(binding, "_calls", None)
    assert route(len(sizes), sum(sizes), I, K, 2 if km else 0) == 1
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        runs = [gg.grouped_gemm_swiglu(*dev, want_act=True, sa_kmajor=km) for _ in range(4)]
        runs.append((*gg.grouped_gemm_swiglu(*dev, sa_kmajor=km)[:2], want[2]))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = gg.grouped_gemm_swiglu(*dev, want_act=True, sa_kmajor=km)
    for _ in range(3):
        for t in captured:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        runs.append(tuple(t.clone() for t in captured))
    for A2, SA2, act in runs:
        assert torch.equal(A2, want[0]) and torch.equal(SA2, want[1]) and torch.equal(act.view(torch.int16), want[2].view(torch.int16))


@pytest.mark.gpu
@pytest.mark.parametrize("km", [False, True])
@pytest.mark.parametrize("native", [True, False])
def test_rows_of_no_group(km, native, monkeypatch):
    """Offsets that leave rows out in front and behind: with fresh outputs (two launches) the groups' rows are those of the one launch, in a
    caller's own outputs (one launch) the other rows stay as they were."""
    sizes, I, K = [0, 3, 17, 1], 640, 1152
    dev = problem([4] + sizes + [9], I, K, 5)              # rows, weights
    dev[2], dev[3] = dev[2][1:5], dev[3][1:5]
    dev[4] = dev[4][1:6].contiguous()                      # [4, 4, 7, 24, 25] of 34 rows
    if km:
        dev[1] = dev[1].t().contiguous()
    if not native:
        monkeypatch.setattr(binding, "_calls", None)
    assert route(4, 34, I, K, 2 if km else 0) == 1
    A2 = torch.full((34, I), 0xAB, dtype=torch.uint8, device=DEV)
    SA2 = torch.full((I // 128, 34) if km else (34, I // 128), -7.0, device=DEV)
    act = torch.full((34, I), 3.0, dtype=torch.bfloat16, device=DEV)
    gg.grouped_gemm_swiglu(*dev, A2=A2, SA2=SA2, act_out=act, sa_kmajor=km)
    fresh = gg.grouped_gemm_swiglu(*dev, want_act=True, sa_kmajor=km)
    rows = lambda t: t.t() if km and t.dtype == torch.float32 else t
    for own, other, mark in zip((A2, SA2, act), fresh, (0xAB, -7.0, 3.0)):
        bits = {1: torch.uint8, 2: torch.int16, 4: torch.int32}[own.element_size()]
        assert torch.equal(rows(own)[4:25].contiguous().view(bits), rows(other)[4:25].contiguous().view(bits))
        assert (rows(own)[:4] == mark).all() and (rows(own)[25:] == mark).all()


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
def test_no_room_for_the_intermediate(native, monkeypatch):
    dev = problem([32] * 256, 1024, 512, 3)
    assert route(256, 8192, 1024, 512) == 1                # 32 MB of intermediate, 8 MB of bytes
    if not native:
        monkeypatch.setattr(binding, "_calls", None)
    want = gg.grouped_gemm_swiglu(*dev)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    room = torch.empty(8 << 20, dtype=torch.uint8, device=DEV)      # for the bytes, 20 MB as the allocator takes them
    limit = torch.cuda.memory_reserved() + (4 << 20)
    torch.cuda.set_per_process_memory_fraction(limit / torch.cuda.get_device_properties(0).total_memory)
    held = []
    try:
        with pytest.raises(torch.OutOfMemoryError):        # what earlier tests left free in pieces of 32 MB
            while len(held) < 1000:
                held.append(torch.empty(32 << 20, dtype=torch.uint8, device=DEV))
        del room
        got = gg.grouped_gemm_swiglu(*dev)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])

"""The binding's native calls (csrc/gg_calls.cpp): what they leave to the Python code, and that both give the same."""
import ctypes

import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

import paper_2508_16584_amd as gg
from paper_2508_16584_amd import binding
from workloads import CONFIGS, make_problem


class Seen(TorchDispatchMode):
    """Notes the operations that it sees."""

    def __init__(self):
        super().__init__()
        self.ops = []

    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        self.ops.append(str(func))
        return func(*args, **(kwargs or {}))


def operands(dev):
    p = make_problem(CONFIGS["tiny"])
    return [p[k].to(dev) for k in ("A", "SA", "B", "SB", "group_offsets")]


def calls():
    binding.load_library()
    assert binding._calls is not None, "csrc/gg_calls.cpp is not built"
    return binding._calls


def test_not_on_the_gpu_is_left_alone():
    c, ops = calls(), operands("cpu")
    X = torch.zeros(8, 256, dtype=torch.bfloat16)
    assert c.grouped_gemm(*ops, False, False) is None
    assert c.grouped_gemm_swiglu(*ops, False, False) is None
    assert c.grouped_gemm_wgrad(ops[0], ops[1], ops[0], ops[1], ops[4], False) is None
    assert c.quantize_rows(X, None, False) is None and c.quantize_cols(X, None) is None
    assert c.swiglu_quantize_rows(X, False, False) is None
    assert c.grouped_gemm(None, 1, "B", ops, X, False, False) is None
    with pytest.raises(TypeError):
        c.quantize_cols(X)
    with pytest.raises(ValueError, match="GPU"):
        gg.quantize_cols(X)


@pytest.mark.parametrize("failure", [FileNotFoundError("g++"), RuntimeError("g++ failed")])
def test_a_build_that_fails_leaves_the_python_code(monkeypatch, tmp_path, failure):
    def run(cmd, verbose):
        raise failure

    old = tmp_path / "calls.so"
    old.write_bytes(b"of another source")
    monkeypatch.setattr(binding, "calls_path", lambda: str(old))
    monkeypatch.setattr(binding, "_run", run)
    with pytest.warns(UserWarning, match="not built"):
        binding._build_calls(False)
    assert not old.exists()


def test_a_file_that_does_not_load_leaves_the_python_code(monkeypatch, tmp_path):
    bad = tmp_path / "calls.so"
    bad.write_bytes(b"no library")
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_calls", None)
    monkeypatch.setattr(binding, "calls_path", lambda: str(bad))
    with pytest.warns(UserWarning, match="not used"):
        binding.load_library()
    assert binding._calls is None and gg.num_variants() > 0


@pytest.mark.gpu
def test_left_to_the_python_code():
    c, (A, SA, B, SB, off) = calls(), operands("cuda")

    class Sub(torch.Tensor):
        pass

    ok = dict(A=A, SA=SA, B=B, SB=SB, off=off, f16=False, km=False)
    wrong = [dict(A=A.as_subclass(Sub)), dict(A=A.to(torch.int8)), dict(A=A[:, :-16]), dict(A=A.t().contiguous().t()), dict(A=A[None]),
             dict(SA=SA[:-1]), dict(SA=SA.cpu()), dict(SA=SA.double()), dict(B=B[:, :-8]), dict(SB=SB[:-1]), dict(off=off[:-1]),
             dict(off=off.long()), dict(km=True), dict(km=1), dict(f16=None)]
    for w in wrong:
        assert c.grouped_gemm(*{**ok, **w}.values()) is None, w
    assert c.grouped_gemm(*ok.values()) is not None
    with torch.device("cuda"):                                  # a mode that sees calls, not operations
        assert c.grouped_gemm(*ok.values()) is None
    with Seen() as seen:
        assert c.grouped_gemm(*ok.values()) is None
        gg.grouped_gemm(A, SA, B, SB, off)
    assert any("empty" in op for op in seen.ops)
    with torch.inference_mode():
        assert gg.grouped_gemm(A, SA, B, SB, off).is_inference()
    X = torch.zeros(8, 200, dtype=torch.bfloat16, device="cuda")
    assert c.quantize_rows(X, None, False) is None              # the library refuses it
    with pytest.raises(gg.GGError):
        gg.quantize_rows(X)


@pytest.mark.gpu
@pytest.mark.parametrize("km", [False, True])
def test_both_routes_give_the_same(km, monkeypatch):
    A, SA, B, SB, off = operands("cuda")
    M, K = 304, 256
    tokens = torch.tensor([0, 100, 100, M], dtype=torch.int32, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(5)
    X = torch.randn(M, K, generator=gen, device="cuda").bfloat16()
    src = torch.randperm(M, generator=gen, device="cuda").int()
    S = SA.t().contiguous() if km else SA
    W, SW = torch.randint(0, 0x78, (3, 256, 384), dtype=torch.uint8, generator=gen, device="cuda"), torch.ones(3, 2, 3, device="cuda")

    def run():
        out = [gg.grouped_gemm(A, S, B, SB, off, sa_kmajor=km), gg.grouped_gemm(A, S, B, SB, off, out_dtype=torch.float16, sa_kmajor=km)]
        out += gg.quantize_rows(X, src, sa_kmajor=km) + gg.quantize_rows(X[:0], sa_kmajor=km)
        out += gg.swiglu_quantize_rows(X, want_act=True, sa_kmajor=km)
        assert gg.swiglu_quantize_rows(X, sa_kmajor=km)[2] is None
        XT, SX = gg.quantize_cols(X, src)
        out += [XT, SX, *gg.quantize_cols(X)]
        out += [gg.grouped_gemm_wgrad(XT, SX, XT, SX, tokens, out_bf16=km)]
        H = torch.cat([X, X[:, :128]], dim=1)                   # the fused kernel takes three blocks of K and more
        out += gg.grouped_gemm_swiglu(*gg.quantize_rows(H, sa_kmajor=km), W, SW, tokens, want_act=True, sa_kmajor=km)
        return out

    for stream in (torch.cuda.current_stream(), torch.cuda.Stream()):
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            calls()
            fast = run()
            with monkeypatch.context() as m:
                m.setattr(binding, "_calls", None)
                slow = run()
        stream.synchronize()
        assert len(fast) == len(slow) and fast[0].dtype == torch.bfloat16 and fast[1].dtype == torch.float16
        for a, b in zip(fast, slow):
            assert a.dtype == b.dtype and a.shape == b.shape and a.device == b.device and torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.gpu
def test_an_error_of_the_runtime_is_raised_and_the_call_made_once():
    """A library whose functions report an error of the HIP runtime (nothing is launched): the status reaches the caller, and the
    Python code, which has the real library, does not make the call again."""
    c, ops = calls(), operands("cuda")
    made = []

    def fake(*types):
        return ctypes.CFUNCTYPE(ctypes.c_int, *types)(lambda *args: made.append(len(args)) or 5)

    vp, i32, i64, u32 = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64, ctypes.c_uint
    fakes = [fake(*[vp] * 6, i32, i64, i32, i32, vp, ctypes.c_size_t, vp, i32, u32), fake(*[vp] * 8, i32, i64, i32, i32, vp, i32, u32),
             fake(*[vp] * 6, i32, i64, i32, i32, vp, u32), fake(*[vp] * 4, i64, i64, i32, vp, u32), fake(*[vp] * 4, i64, i64, i32, vp),
             fake(*[vp] * 4, i64, i32, vp, u32)]
    A, SA, B, SB, off = ops
    X = torch.zeros(32, 256, dtype=torch.bfloat16, device="cuda")
    XT, SX = gg.quantize_cols(X)
    runs = [lambda: gg.grouped_gemm(*ops), lambda: gg.grouped_gemm_swiglu(*ops), lambda: gg.grouped_gemm_wgrad(XT, SX, XT, SX, off),
            lambda: gg.quantize_rows(X), lambda: gg.quantize_cols(X), lambda: gg.swiglu_quantize_rows(X)]
    try:
        c.bind(*(ctypes.cast(f, vp).value for f in fakes), binding._check)
        for i, run in enumerate(runs):
            with pytest.raises(gg.GGError) as e:
                run()
            assert e.value.status == 5 and len(made) == i + 1
    finally:
        binding._load_calls(binding.load_library())

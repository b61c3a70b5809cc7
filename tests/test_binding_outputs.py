"""Outputs that a caller hands in: one of another shape than the kernels write is refused before the library is called.
No GPU: host tensors that report themselves as device tensors, and a library that only records its calls."""
import types

import pytest
import torch

import paper_2508_16584_amd as gg
from paper_2508_16584_amd import binding


class DeviceTensor(torch.Tensor):
    is_cuda = True


def dev(*shape, dtype=torch.uint8):
    return torch.zeros(shape, dtype=dtype).as_subclass(DeviceTensor)


def f32(*shape):
    return dev(*shape, dtype=torch.float32)


def bf16(*shape):
    return dev(*shape, dtype=torch.bfloat16)


def i32(*shape):
    return dev(*shape, dtype=torch.int32)


class RecordingLibrary:
    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            self.calls.append(name)
            return 0
        return call


@pytest.fixture
def library(monkeypatch):
    lib = RecordingLibrary()
    monkeypatch.setattr(binding, "load_library", lambda: lib)
    return lib


STREAM = types.SimpleNamespace(cuda_stream=0)
M, I, K, G = 48, 256, 384, 2


# (the call, its outputs: name -> the tensor that fits)
CASES = {
    "swiglu_quantize_rows": (lambda **o: gg.swiglu_quantize_rows(bf16(M, 2 * I), stream=STREAM, **o),
                             dict(A=lambda: dev(M, I), SA=lambda: f32(M, I // 128), act_out=lambda: bf16(M, I))),
    "swiglu_quantize_rows K-block-major": (lambda **o: gg.swiglu_quantize_rows(bf16(M, 2 * I), stream=STREAM, sa_kmajor=True, **o),
                                           dict(A=lambda: dev(M, I), SA=lambda: f32(I // 128, M), act_out=lambda: bf16(M, I))),
    "quantize_rows": (lambda **o: gg.quantize_rows(bf16(M, K), stream=STREAM, **o),
                      dict(A=lambda: dev(M, K), SA=lambda: f32(M, K // 128))),
    "quantize_cols": (lambda **o: gg.quantize_cols(bf16(M, K), stream=STREAM, **o),
                      dict(XT=lambda: dev(K, M), SX=lambda: f32(1, K))),
    "grouped_gemm_swiglu": (lambda **o: gg.grouped_gemm_swiglu(dev(M, K), f32(M, 3), dev(G, 2 * I, K), f32(G, 4, 3), i32(G + 1), stream=STREAM, **o),
                            dict(A2=lambda: dev(M, I), SA2=lambda: f32(M, I // 128), act_out=lambda: bf16(M, I))),
    "grouped_gemm_wgrad": (lambda **o: gg.grouped_gemm_wgrad(dev(K, M), f32(1, K), dev(I, M), f32(1, I), i32(G + 1), stream=STREAM, **o),
                           dict(dW=lambda: f32(G, I, K))),
    "grouped_gemm": (lambda **o: gg.grouped_gemm(dev(M, K), f32(M, 3), dev(G, I, K), f32(G, 2, 3), i32(G + 1), stream=STREAM, **o),
                     dict(C=lambda: bf16(M, I))),
}


@pytest.mark.parametrize("case", CASES)
def test_an_output_of_another_shape_is_refused(library, case):
    call, outputs = CASES[case]
    call(**{name: make() for name, make in outputs.items()})
    assert len(library.calls) == 1
    for name, make in outputs.items():
        fits = make()
        for dim in range(fits.dim()):
            for size in (fits.shape[dim] - 1, fits.shape[dim] + 1, 0):
                shape = list(fits.shape)
                shape[dim] = size
                library.calls.clear()
                with pytest.raises(ValueError):
                    call(**{name: dev(*shape, dtype=fits.dtype)})
                assert not library.calls, f"{name} {shape}"


# The padded path: rows past the problem's are left alone, so there may be more of them, but not fewer, and no other width.
PADDED = {
    "grouped_gemm_padded": lambda rows, cols, km=False: gg.grouped_gemm_padded(
        dev(M, K), f32(3, M) if km else f32(M, 3), dev(G, I, K), f32(G, 2, 3), i32(G + 1), C_pad=bf16(rows, cols), stream=STREAM, sa_kmajor=km),
    "grouped_gemm_padded K-block-major": lambda rows, cols: PADDED["grouped_gemm_padded"](rows, cols, True),
    "unpad": lambda rows, cols: gg.unpad(bf16(2 * M, I), i32(G + 1), i32(G + 1), M, C=bf16(rows, cols), stream=STREAM),
}


@pytest.mark.parametrize("case", PADDED)
def test_the_padded_path_refuses_an_output_that_is_too_small(library, case):
    for rows in (M, M + 1, 3 * M):
        PADDED[case](rows, I)
    done = len(library.calls)
    for rows, cols in ((M - 1, I), (0, I), (M, I - 8), (M, I + 8), (M, 0)):
        with pytest.raises(ValueError):
            PADDED[case](rows, cols)
    with pytest.raises(ValueError):
        gg.unpad(bf16(2 * M, I), i32(G + 1), i32(G), M, stream=STREAM)        # offsets of another number of groups
    assert len(library.calls) == done

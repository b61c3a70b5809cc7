"""The calls whose speed counts, over the range of sizes and options that they are used with.

Each case is one use of the library through its public entry points, as the README shows them:
  gemm      the grouped GEMM alone: grouped_gemm on operands that are at hand
  mlp       the forward pass of an expert MLP: quantize_rows through the routing permutation, the first GEMM, the
            activation with its quantiser (two calls, or one with grouped_gemm_swiglu), the second GEMM
  wgrad     the weight-gradient GEMM alone: grouped_gemm_wgrad
  layer     one expert layer in training: forward, input gradient and weight gradient with all their quantisers
  operands  what a training step makes of one activation tensor: its row-quantised form for the forward GEMM and its
            column-quantised form for the weight gradient
G experts share N and K (mlp: K the hidden and I the intermediate size), M rows are routed to them by `law`.
"""
import numpy as np
import torch

import paper_2508_16584_amd as gg

DEV = "cuda:0"


def listed():
    return [
        # the smallest problem of this repository (workload "tiny"): launch and host latency
        dict(name="tiny", op="gemm", G=4, M=600, N=256, K=256, law="uniform", kmajor=False, out="bf16"),
        # one decoding step of 32 sequences, top-2 routing over the 8 experts of a GPU: a few rows per expert
        dict(name="decode_step", op="mlp", G=8, M=64, T=32, K=7168, I=2048, law="uniform", kmajor=False, fused=False),
        # workload "decode": 2048 rows over 64 experts, some without rows; the weights dominate the bytes
        dict(name="decode", op="gemm", G=64, M=2048, N=4096, K=7168, law="dirichlet0.3", kmajor=False, out="bf16"),
        # nothing a multiple of a tile or of a scale block, binary16 output
        dict(name="ragged", op="gemm", G=8, M=3001, N=4104, K=7232, law="dirichlet1", kmajor=False, out="f16"),
        # workload "gate_up": first projection in prefill or training, the headline of the benchmark
        dict(name="gate_up", op="gemm", G=8, M=8192, N=4096, K=7168, law="dirichlet1", kmajor=False, out="bf16"),
        # workload "down": second projection, strongly skewed expert popularity, K-block-major scales
        dict(name="down", op="gemm", G=32, M=16384, N=7168, K=2048, law="zipf", kmajor=True, out="bf16"),
        # workload "many_small": 256 experts with about 128 rows each
        dict(name="many_small", op="gemm", G=256, M=32768, N=4096, K=7168, law="poisson", kmajor=False, out="bf16"),
        # the forward pass of gate_up's MLP in three calls, the activation in the first GEMM
        dict(name="mlp", op="mlp", G=8, M=8192, T=8192, K=7168, I=2048, law="dirichlet1", kmajor=True, fused=True),
        # the weight gradient of gate_up's layer, fp32 gradients
        dict(name="wgrad", op="wgrad", G=8, M=8192, N=4096, K=7168, law="dirichlet1", out="f32"),
        # the weight gradient of many experts with few tokens each, bfloat16 gradients
        dict(name="wgrad_short", op="wgrad", G=64, M=2048, N=4096, K=7168, law="dirichlet0.3", out="bf16"),
        # a small layer, forward and backward, with sizes that are no multiple of a tile
        dict(name="layer", op="layer", G=5, M=1264, T=640, N=768, K=1280, law="dirichlet1", out="f32"),
        # both quantised forms of a large activation tensor, gathered through a top-2 routing
        dict(name="operands", op="operands", M=16384, T=8192, K=7168),
    ]


def _log_int(rng, lo, hi, step=1):
    """An integer multiple of step in [lo, hi], spread over the logarithm of the range."""
    v = lo * (hi / lo) ** rng.random()
    return min(hi, max(lo, int(round(v / step)) * step))


LAWS = ("uniform", "dirichlet1", "dirichlet0.3", "zipf", "poisson")
MAX_BYTES, MAX_FLOPS = 4.0e9, 5.5e11      # of a drawn case: under the largest listed ones


def draw(rng):
    while True:
        op = rng.choice(("gemm", "gemm", "gemm", "mlp", "mlp", "wgrad", "layer", "operands"))
        case = dict(op=op)
        if op == "operands":
            case.update(K=_log_int(rng, 256, 8192, 128), T=_log_int(rng, 16, 16384))
            case["M"] = max(16, case["T"] * rng.randint(1, 2) // 16 * 16)
        else:
            case.update(G=_log_int(rng, 1, 256), law=rng.choice(LAWS))
            if op == "gemm":
                ragged = rng.random() < 0.25
                case.update(M=_log_int(rng, 1, 32768), N=_log_int(rng, 256, 8192, 8 if ragged else 128),
                            K=_log_int(rng, 256, 8192, 16 if ragged else 128),
                            kmajor=rng.random() < 0.4, out="f16" if rng.random() < 0.2 else "bf16")
            elif op == "mlp":
                top = rng.choice((1, 2, 4, 8))
                case.update(T=_log_int(rng, 1, 8192), K=_log_int(rng, 512, 8192, 128), I=_log_int(rng, 256, 4096, 128),
                            kmajor=rng.random() < 0.4, fused=rng.random() < 0.5)
                case["M"] = case["T"] * top
            else:
                case.update(M=_log_int(rng, 16, 16384, 16), N=_log_int(rng, 256, 8192, 256 if op == "layer" else 128),
                            K=_log_int(rng, 256, 8192, 256), out="bf16" if rng.random() < 0.4 else "f32")
                if op == "layer":
                    case["T"] = max(1, case["M"] // rng.choice((1, 2, 4)))
        w = work(case)
        if w["bytes"] <= MAX_BYTES and w["flops"] <= MAX_FLOPS:
            return case


# ---------------------------------------------------------------------------------------------- inputs
def _sizes(case):
    """Rows per expert: fixed by the case, so that every pass does the same work (prepare deals them to the experts)."""
    G, M, law = case["G"], case["M"], case["law"]
    rng = np.random.default_rng([G, M, case["K"], LAWS.index(law)])
    if law == "uniform":
        p = rng.random(G) + 1e-3
    elif law.startswith("dirichlet"):
        p = rng.dirichlet(np.full(G, float(law[len("dirichlet"):]))) + 1e-9
    elif law == "zipf":
        p = np.arange(1, G + 1, dtype=np.float64) ** -1.1
    else:
        p = rng.poisson(128, G) + 1e-3
    return rng.multinomial(M, p / p.sum())


def _offsets(case, rng):
    sizes = rng.permutation(_sizes(case))
    return torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)).to(DEV)


def _scaled_e4m3(x, amax):
    scale = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
    return (x / scale).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8), scale


def _quantised_rows(rows, cols, std, gen):
    """e4m3 [rows, cols] of normal values and one scale per row and 128 columns; the last block may be short."""
    kb = -(-cols // 128)
    q = torch.empty((rows, cols), dtype=torch.uint8, device=DEV)
    s = torch.empty((rows, kb), dtype=torch.float32, device=DEV)
    for r in range(0, rows, 8192):
        n = min(8192, rows - r)
        x = torch.randn((n, kb * 128), generator=gen, device=DEV) * std
        x[:, cols:] = 0
        x = x.view(n, kb, 128)
        b, c = _scaled_e4m3(x, x.abs().amax(dim=2, keepdim=True))
        q[r:r + n] = b.view(n, kb * 128)[:, :cols]
        s[r:r + n] = c.view(n, kb)
    return q, s


def _weights(G, N, K, gen):
    """e4m3 [G, N, K] and one scale per 128 x 128 block; the last blocks may be short."""
    nb, kb = -(-N // 128), -(-K // 128)
    q = torch.empty((G, N, K), dtype=torch.uint8, device=DEV)
    s = torch.empty((G, nb, kb), dtype=torch.float32, device=DEV)
    for g in range(G):
        x = torch.randn((nb * 128, kb * 128), generator=gen, device=DEV) * 0.02
        x[N:] = 0
        x[:, K:] = 0
        x = x.view(nb, 128, kb, 128)
        b, c = _scaled_e4m3(x, x.abs().amax(dim=3, keepdim=True).amax(dim=1, keepdim=True))
        q[g] = b.view(nb * 128, kb * 128)[:N, :K]
        s[g] = c.view(nb, kb)
    return q, s


def _transposed_weights(q, s):
    return q.transpose(1, 2).contiguous(), s.transpose(1, 2).contiguous()


def _routing(case, rng):
    """Token of every routed row: each token appears about M / T times, in random order."""
    src = np.concatenate([rng.permutation(case["T"]) for _ in range(-(-case["M"] // case["T"]))])[:case["M"]]
    return torch.from_numpy(src.astype(np.int32)).to(DEV)


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    rng = np.random.default_rng(seed)
    op, st = case["op"], dict(case=case)
    if op != "operands":
        st["off"] = _offsets(case, rng)
    if op == "gemm":
        st["A"], st["SA"] = _quantised_rows(case["M"], case["K"], 1.0, gen)
        if case["kmajor"]:
            st["SA"] = st["SA"].t().contiguous()
        st["B"], st["SB"] = _weights(case["G"], case["N"], case["K"], gen)
    elif op == "mlp":
        st["X"] = torch.randn((case["T"], case["K"]), generator=gen, device=DEV).to(torch.bfloat16)
        st["src"] = _routing(case, rng)
        st["W1"], st["S1"] = _weights(case["G"], 2 * case["I"], case["K"], gen)
        st["W2"], st["S2"] = _weights(case["G"], case["K"], case["I"], gen)
    elif op == "wgrad":
        st["XT"], sx = _quantised_rows(case["K"], case["M"], 1.0, gen)
        st["DYT"], sdy = _quantised_rows(case["N"], case["M"], 0.02, gen)
        st["SX"], st["SDY"] = sx.t().contiguous(), sdy.t().contiguous()
    elif op == "layer":
        st["X"] = torch.randn((case["T"], case["K"]), generator=gen, device=DEV).to(torch.bfloat16)
        st["dY"] = (torch.randn((case["M"], case["N"]), generator=gen, device=DEV) * 0.02).to(torch.bfloat16)
        st["src"] = _routing(case, rng)
        st["W"], st["SW"] = _weights(case["G"], case["N"], case["K"], gen)
        st["Wt"], st["SWt"] = _transposed_weights(st["W"], st["SW"])
    else:
        st["X"] = torch.randn((case["T"], case["K"]), generator=gen, device=DEV).to(torch.bfloat16)
        st["src"] = _routing(case, rng)
    return st


# ---------------------------------------------------------------------------------------------- one pass
def run(st):
    case = st["case"]
    op = case["op"]
    if op == "gemm":
        return gg.grouped_gemm(st["A"], st["SA"], st["B"], st["SB"], st["off"], sa_kmajor=case["kmajor"],
                               out_dtype=torch.float16 if case["out"] == "f16" else torch.bfloat16)
    if op == "mlp":
        km = case["kmajor"]
        A, SA = gg.quantize_rows(st["X"], st["src"], sa_kmajor=km)
        if case["fused"]:
            A2, SA2, _ = gg.grouped_gemm_swiglu(A, SA, st["W1"], st["S1"], st["off"], sa_kmajor=km)
        else:
            H = gg.grouped_gemm(A, SA, st["W1"], st["S1"], st["off"], sa_kmajor=km)
            A2, SA2, _ = gg.swiglu_quantize_rows(H, sa_kmajor=km)
        return gg.grouped_gemm(A2, SA2, st["W2"], st["S2"], st["off"], sa_kmajor=km)
    if op == "wgrad":
        return gg.grouped_gemm_wgrad(st["XT"], st["SX"], st["DYT"], st["SDY"], st["off"], out_bf16=case["out"] == "bf16")
    if op == "layer":
        A, SA = gg.quantize_rows(st["X"], st["src"])
        Y = gg.grouped_gemm(A, SA, st["W"], st["SW"], st["off"])
        dA, SdA = gg.quantize_rows(st["dY"])
        dX = gg.grouped_gemm(dA, SdA, st["Wt"], st["SWt"], st["off"])
        XT, SX = gg.quantize_cols(st["X"], st["src"])
        DYT, SDY = gg.quantize_cols(st["dY"])
        dW = gg.grouped_gemm_wgrad(XT, SX, DYT, SDY, st["off"], out_bf16=case["out"] == "bf16")
        return Y, dX, dW
    A, SA = gg.quantize_rows(st["X"], st["src"])
    XT, SX = gg.quantize_cols(st["X"], st["src"])
    return A, SA, XT, SX


# ---------------------------------------------------------------------------------------------- what it cannot do without
def work(case):
    op, M, K = case["op"], case["M"], case["K"]
    if op == "operands":
        return dict(bytes=2 * case["T"] * K + 4 * M + 2 * (M * K + 4 * M * K // 128), flops=0)
    G, sizes = case["G"], _sizes(case)
    used = int((sizes > 0).sum())             # experts without rows: their weights are never read

    def weights(n, k):
        return used * (n * k + 4 * (-(-n // 128)) * (-(-k // 128)))

    def rows(k):
        return M * (k + 4 * (-(-k // 128)))
    if op == "gemm":
        N = case["N"]
        return dict(bytes=rows(K) + weights(N, K) + 2 * M * N, flops=2 * M * N * K)
    if op == "mlp":
        n1 = 2 * case["I"]
        return dict(bytes=2 * case["T"] * K + 4 * M + weights(n1, K) + weights(K, case["I"]) + 2 * M * K,
                    flops=2 * M * K * (n1 + case["I"]))
    N = case["N"]
    out = G * N * K * (2 if case["out"] == "bf16" else 4)
    if op == "wgrad":
        return dict(bytes=(K + N) * (M + 4 * (-(-M // 128))) + out, flops=2 * M * N * K)
    return dict(bytes=2 * case["T"] * K + 2 * M * N + 4 * M + weights(N, K) + weights(K, N) + 2 * M * (N + K) + out,
                flops=6 * M * N * K)


# Four times what this path shows against its own definition with the sums in 64 bits (the last factor for "max" is two
# where it is one step of the output format).  The FP8 matrix instruction truncates inside a block of products, which
# is all that separates fp32 results from the definition (1.35e-5) and what moves 1 % of the bfloat16 results and 6 % of
# the binary16 results by a step (2.3e-4, 8e-5); in the MLP such a step moves bytes of the second operand (2.3e-3).
TOLERANCE = {
    "f32": {"rel": 6e-5, "max": 4.5e-4},
    "bf16": {"rel": 1e-3, "max": 0.016},
    "f16": {"rel": 3.5e-4, "max": 0.002},
    "mlp": {"rel": 9e-3, "max": 0.27},
    "layer": {"rel": 1e-3, "max": 0.016},      # two bfloat16 results and the weight gradient
    "operands": "exact",                       # the quantisers are defined bit for bit
}


def tolerance(case):
    return TOLERANCE[case["op"] if case["op"] in TOLERANCE else case["out"]]

#!/usr/bin/env python3
"""Benchmark of the padding-free FP8 grouped GEMM (libgg_fp8) on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload gate_up] [--variant -1]

A step is one pass of the whole hot path over one batch of synthetic input: one
gg_fp8_grouped_gemm call (tile schedule from the device-resident group offsets, bounded operand
fetch, FP8 MFMA contraction, fused block-scale dequantisation, bf16 bounded store).  Inputs are
resident in HBM before the timed region; the steps rotate over several copies of the input so
that the 256 MB Infinity Cache does not serve them.  The metric is FP8 TFLOP/s on valid rows,
2 * M_total * N * K / time.  One JSON line is printed; besides the contract fields it carries
  roofline      the GEMM kernel against the FP8 MFMA (or HBM) roofline, from per-launch HIP events,
  cpu_baseline  the CPU oracle timed on a bounded row sample of the same workload,
  pad_path      the pad-then-GEMM comparison of the paper (Sec. 3) on the same inputs: time,
                speed-up of the padding-free path, memory saved.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

FP8_MFMA_PEAK_TFLOPS = 5033.0     # MI355X dense FP8: 256 CU x 8192 flop/clk/CU x 2.4 GHz
HBM_PEAK_GBS = 8000.0             # MI355X HBM3E

TRAFFIC_TABLE = os.path.join(ROOT, "profiles", "hbm_traffic.md")


def profiled_traffic(op, workload, layout, kernel):
    """HBM bytes per launch from the table under profiles/ that earlier rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of
    this script wrote (each row: op, workload, scale layout, kernel, read bytes, written bytes, total; the file gives
    the commands and the copy-kernel calibration).  It is NOT a measurement of the present run: the JSON line says so
    in `traffic_source`, and a row is only used when it was taken with the same kernel variant.  None if there is
    no such row."""
    try:
        with open(TRAFFIC_TABLE) as f:
            for line in f:
                c = [x.strip().strip("`") for x in line.strip().strip("|").split("|")]
                if len(c) >= 7 and c[0] == op and c[1] == workload and c[2] == layout and c[3] == kernel:
                    return int(c[6])
    except (OSError, ValueError):
        pass
    return None


TRAFFIC_SOURCE = "profiles/hbm_traffic.md: rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of this command on an earlier box, not this run"


def clock_warmup(step, ms):
    """Untimed launches of the benchmarked step for about `ms` milliseconds, ahead of the W warm-up steps: after an
    idle period the GPU needs some 30 ms of load to reach its sustained clock (the first 100 launches of gate_up fall
    from 277 to 246 us each), and W launches of a 0.3 ms kernel end well inside that ramp.  Returns the launch count."""
    import torch
    n, t0 = 0, time.perf_counter()
    while ms > 0:
        for _ in range(10):
            step(n)
            n += 1
        torch.cuda.synchronize()
        if (time.perf_counter() - t0) * 1e3 >= ms:
            break
    return n


def timed_region(step, steps):
    """Exactly `steps` launches back to back between two synchronisations.  Returns (wall-clock ms per step, ms per
    step between two HIP events recorded on the launch stream around the region): the second is the kernel's average
    launch duration as the stream sees it, gaps between launches included."""
    import torch
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    e0.record()                    # HIP events on the stream the kernel is launched on (torch's current stream)
    for i in range(steps):
        step(i)
    e1.record()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    return wall * 1e3 / steps, e0.elapsed_time(e1) / steps


def per_launch_ms(step, steps):
    """The same launches again, each between its own pair of HIP events (untimed for the headline: the event pairs
    keep consecutive launches apart and add a few microseconds each): for median, minimum and maximum."""
    import numpy as np
    import torch
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
    for i in range(steps):
        ev[i][0].record()
        step(i)
        ev[i][1].record()
    torch.cuda.synchronize()
    return np.array([a.elapsed_time(b) for a, b in ev])


def algorithmic_bytes(sizes, N, K):
    """A + SA + B (non-empty groups only) + SB + C, each touched once."""
    import numpy as np
    M = int(np.sum(sizes))
    nonempty = int(np.sum(np.asarray(sizes) > 0))
    KB, NB = K // 128, N // 128
    return M * K + M * KB * 4 + nonempty * N * K + nonempty * NB * KB * 4 + M * N * 2




def copy_calibration(dev):
    """A plain device copy of known size (reads 1 GiB, writes 1 GiB), for scaling FETCH_SIZE / WRITE_SIZE."""
    import torch
    src = torch.empty(1 << 30, dtype=torch.uint8, device=dev).random_(0, 255)
    dst = torch.empty_like(src)
    for _ in range(3):
        dst.copy_(src)
    torch.cuda.synchronize()
    del src, dst


def bench_quantize_rows(args, cfg, dev):
    """quantize_rows: bf16 activations [M_total, K] of the workload -> e4m3 + 1x128 scales, gathered by a routing
    permutation (2K bytes read, K + 4K/128 written per row, plus 4 bytes of index).
    swiglu_quantize_rows: the workload's GEMM output [M_total, N] bf16 (gate | up) -> e4m3 [M_total, N/2] + scales
    (2N bytes read, N/2 + 4(N/2)/128 written per row).
    quantize_cols: the same activations -> XT [K, M_total] e4m3 + [M_total/128, K] scales, quantised along the tokens
    and transposed (the producer of the weight-gradient GEMM's operands; the same bytes per row).  All HBM-bound."""
    import numpy as np
    import torch

    import paper_2508_16584_amd as gg
    from workloads import group_sizes

    fused = args.op == "swiglu_quantize_rows"
    cols = args.op == "quantize_cols"
    km = args.sa_layout == "kmajor" and not cols
    sizes = group_sizes(cfg, cfg.seed)
    M = int(np.sum(sizes))
    width_in = cfg.N if fused else cfg.K                      # columns of the bf16 input
    width_out = cfg.N // 2 if fused else cfg.K                # columns of the e4m3 output
    gen = torch.Generator(device=dev)
    gen.manual_seed(cfg.seed)
    alg_bytes = M * (2 * width_in + width_out + 4 * (width_out // 128) + (0 if fused else 4))
    copies = args.copies or max(2, min(8, int(np.ceil(1.0e9 / alg_bytes))))
    rng = np.random.default_rng(cfg.seed)
    sets = []
    for _ in range(copies):
        X = (torch.randn((M, width_in), generator=gen, device=dev, dtype=torch.float32) * (1.7 if fused else 1.0)).to(torch.bfloat16)
        src = None if fused else torch.from_numpy(rng.permutation(M).astype(np.int32)).to(dev)
        if cols:
            sets.append((X, src, torch.empty((width_out, M), dtype=torch.uint8, device=dev),
                         torch.empty(((M + 127) // 128, width_out), dtype=torch.float32, device=dev)))
            continue
        sets.append((X, src, torch.empty((M, width_out), dtype=torch.uint8, device=dev),
                     torch.empty((width_out // 128, M) if km else (M, width_out // 128), dtype=torch.float32, device=dev)))

    def step(i):
        X, src, A, SA = sets[i % copies]
        if fused:
            gg.swiglu_quantize_rows(X, A=A, SA=SA, sa_kmajor=km)
        elif cols:
            gg.quantize_cols(X, src, XT=A, SX=SA)
        else:
            gg.quantize_rows(X, src, A=A, SA=SA, sa_kmajor=km)

    n_ramp = clock_warmup(step, args.clock_warmup_ms)
    for i in range(args.warmup):
        step(i)
    torch.cuda.synchronize()
    ms_per_step, kern_avg_ms = timed_region(step, args.steps)
    kern_ms = per_launch_ms(step, args.steps)
    if args.copy_calibration:
        copy_calibration(dev)
    achieved = alg_bytes / (kern_avg_ms * 1e-3) / 1e9
    kname = "gg_swiglu_quantize_rows_kernel" if fused else "gg_quantize_cols_kernel" if cols else "gg_quantize_rows_kernel"
    traffic = profiled_traffic(args.op, args.workload, args.sa_layout, kname)
    out = {
        "metric": "algorithmic GB/s, " + ("bf16 gate|up rows -> silu(gate)*up -> e4m3 + 1x128 scales" if fused else
                                          "bf16 rows -> e4m3 [K, M_total] + scales per 128 tokens, gathered into group order and transposed" if cols else
                                          "bf16 rows -> e4m3 + 1x128 scales gathered into group order"),
        "value": round(alg_bytes / (ms_per_step * 1e-3) / 1e9, 1), "unit": "GB/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(ms_per_step, 4), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "bf16 in, fp32 arithmetic, e4m3 + fp32 scales out", "data": "synthetic",
        "config": {"workload": args.workload + (" output" if fused else " activations"), "op": args.op, "M_total": M,
                   "columns_in": width_in, "columns_out": width_out, "input_copies_rotated": copies,
                   "clock_warmup_launches": n_ramp,
                   "sa_layout": "block-major [M_total/128, K]" if cols else "K-block-major [K/128, M_total]" if km else "row-major [M_total, K/128]"},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": traffic,
                     "traffic_source": TRAFFIC_SOURCE if traffic is not None else None, "kernel": kname,
                     "kernel_avg_ms": round(kern_avg_ms, 4), "kernel_median_ms": round(float(np.median(kern_ms)), 4),
                     "kernel_min_ms": round(float(kern_ms.min()), 4),
                     "algorithmic_bytes": int(alg_bytes)},
    }
    if not args.no_cpu_baseline:
        from oracle import gg_oracle
        X, src, A, SA = sets[0]
        rows = np.arange(0, M, max(1, M // 4096))[:4096]
        xb = X.view(torch.int16).cpu().numpy().view(np.uint16)
        t0 = time.perf_counter()
        if cols:
            feats = np.arange(0, width_out, max(1, width_out // 1024))[:1024]        # features are independent of each other
            rows = np.arange(M)
            A_ref, SA_ref = gg_oracle.quantize_cols(np.ascontiguousarray(xb[:, feats]), src.cpu().numpy())
        elif fused:
            _, A_ref, SA_ref = gg_oracle.swiglu_quantize_rows(xb[rows])
        else:
            A_ref, SA_ref = gg_oracle.quantize_rows(xb, src.cpu().numpy()[rows])
        cpu_s = time.perf_counter() - t0
        if cols:
            same = float(np.mean(A.cpu().numpy()[feats] == A_ref))
            assert same == 1.0 and np.array_equal(SA.cpu().numpy()[:, feats], SA_ref), "bench.py --op quantize_cols: GPU output differs from the oracle on the sample"
            rows = feats             # for the sample's description below
        else:
            same = float(np.mean(A.cpu().numpy()[rows] == A_ref))
        out["cpu_baseline"] = {"value": round(len(rows) / (width_out if cols else M) * alg_bytes / cpu_s / 1e9, 4), "unit": "GB/s",
                               "cores": 1, "kind": "oracle",
                               "sample": (f"{len(rows)} of the {width_out} features, all tokens" if cols else f"{len(rows)} of the {M} output rows") + f", NumPy oracle, {cpu_s:.1f} s",
                               "gpu_bytes_equal_oracle_on_sample": round(same, 6)}
    print(json.dumps(out))


def wgrad_kernel(G, M, N, K, bf16, SX=None, SDY=None):
    """Name of the kernel that the weight-gradient call launches for these arguments."""
    import paper_2508_16584_amd as gg
    way = gg.wgrad_route(G, M, N, K, bf16, SX, SDY)
    return "gg_wgrad_sq_kernel" if "square" in way else "gg_wgrad_kp_kernel" if "chain" in way else "gg_wgrad_kernel"


def bench_wgrad(args, cfg, dev):
    """wgrad: the variable-K grouped GEMM of training on the workload's layer (gg_fp8_grouped_gemm_wgrad):
    XT [K, M_total], DYT [N, M_total] e4m3 with one scale per row and block of 128 tokens -> dW [G, N, K] fp32, the
    workload's group sizes as token counts.  The output is 4 G N K bytes (939.5 MB on gate_up against 92 MB of
    operands and 96 us of matrix instructions at the datasheet peak): the roofline that bounds it is HBM."""
    import numpy as np
    import torch

    import paper_2508_16584_amd as gg
    from workloads import group_sizes

    sizes = group_sizes(cfg, cfg.seed)
    M = int(np.sum(sizes))
    if M % 16:
        raise SystemExit(f"bench.py --op wgrad: M_total = {M} is not a multiple of 16")
    G, N, K = len(sizes), cfg.N, cfg.K
    MB = (M + 127) // 128
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)).to(dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(cfg.seed)

    def operand(rows, std):
        x = torch.randn((rows, MB * 128), generator=gen, device=dev, dtype=torch.float32) * std
        amax = x.view(rows, MB, 128).abs().amax(dim=2).clamp_min(1e-30)
        scale = amax / 448.0
        q = (x.view(rows, MB, 128) / scale[:, :, None]).clamp(-448, 448).to(torch.float8_e4m3fn)
        return q.view(torch.uint8).view(rows, MB * 128)[:, :M].contiguous(), scale.t().contiguous()

    XT, SX = operand(K, 1.0)
    DYT, SDY = operand(N, 0.02)
    bf16 = args.wgrad_out == "bf16"
    es = 2 if bf16 else 4
    alg_bytes = (K + N) * M + 4 * (K + N) * MB + es * G * N * K
    flops = 2.0 * M * N * K
    copies = args.copies or (2 if es * G * N * K < (4 << 30) else 1)
    outs = [torch.empty((G, N, K), dtype=torch.bfloat16 if bf16 else torch.float32, device=dev) for _ in range(copies)]

    def step(i):
        gg.grouped_gemm_wgrad(XT, SX, DYT, SDY, off, dW=outs[i % copies], out_bf16=bf16)

    n_ramp = clock_warmup(step, args.clock_warmup_ms)
    for i in range(args.warmup):
        step(i)
    torch.cuda.synchronize()
    ms_per_step, kern_avg_ms = timed_region(step, args.steps)
    kern_ms = per_launch_ms(step, args.steps)
    achieved = alg_bytes / (kern_avg_ms * 1e-3) / 1e9
    kernel = wgrad_kernel(G, M, N, K, bf16, SX, SDY)
    wg_traffic = profiled_traffic("wgrad", args.workload, args.wgrad_out, kernel)
    out = {
        "metric": "FP8 TFLOP/s on the tokens of the groups, variable-K grouped GEMM dW^g = dY^g^T X^g (e4m3 operands scaled per "
                  "128 tokens, fp32 accumulate, " + ("bf16" if bf16 else "fp32") + " out)",
        "value": round(flops / (ms_per_step * 1e-3) / 1e12, 2), "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(ms_per_step, 4), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "fp8_e4m3 in, fp32 accumulate, " + ("bf16" if bf16 else "fp32") + " out", "data": "synthetic",
        "config": {"workload": args.workload + " layer, weight gradient", "op": "wgrad", "output": args.wgrad_out, "G": G, "M_total": M, "N": N, "K": K,
                   "tokens_per_group_min_max": [int(sizes.min()), int(sizes.max())], "output_copies_rotated": copies,
                   "clock_warmup_launches": n_ramp},
        "roofline": {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBS, 4), "traffic": wg_traffic,
                     "traffic_source": TRAFFIC_SOURCE if wg_traffic is not None else None, "kernel": kernel,
                     "kernel_avg_ms": round(kern_avg_ms, 4), "kernel_median_ms": round(float(np.median(kern_ms)), 4),
                     "kernel_min_ms": round(float(kern_ms.min()), 4), "algorithmic_bytes": int(alg_bytes),
                     "mfma_frac_of_fp8_peak": round(flops / (kern_avg_ms * 1e-3) / 1e12 / FP8_MFMA_PEAK_TFLOPS, 4)},
    }
    if not args.no_cpu_baseline:
        from oracle import gg_oracle
        rng = np.random.default_rng(cfg.seed)
        n_sel, k_sel = np.sort(rng.choice(N, 256, replace=False)), np.sort(rng.choice(K, 512, replace=False))
        h = lambda t, sel: t[torch.from_numpy(sel).to(dev)].cpu().numpy()
        xt, dyt = h(XT, k_sel), h(DYT, n_sel)
        sx, sdy = SX.cpu().numpy()[:, k_sel], SDY.cpu().numpy()[:, n_sel]
        t0 = time.perf_counter()
        ref = gg_oracle.grouped_gemm_wgrad(xt, sx, dyt, sdy, off.cpu().numpy(), with_abs_sum=True)
        cpu_s = time.perf_counter() - t0
        got = outs[(args.steps - 1) % copies][:, torch.from_numpy(n_sel).to(dev)][:, :, torch.from_numpy(k_sel).to(dev)].float().cpu().numpy()
        err = np.abs(got.astype(np.float64) - ref["D"])
        ulp = gg_oracle.bf16_ulp(ref["D"]) if bf16 else np.spacing(np.abs(ref["D"]).astype(np.float32)).astype(np.float64)
        bound = ulp + 2.0 ** -10 * ref["S"]
        assert np.all(err <= bound), "bench.py --op wgrad: GPU output outside the tolerance of tests/test_gpu_wgrad.py on the oracle's sample"
        out["cpu_baseline"] = {"value": round(2.0 * M * len(n_sel) * len(k_sel) / cpu_s / 1e12, 5), "unit": "TFLOP/s", "cores": os.cpu_count(),
                               "kind": "oracle", "sample": f"{len(n_sel)} rows of dY^T x {len(k_sel)} features of every group, NumPy oracle, {cpu_s:.1f} s",
                               "gpu_bits_equal_oracle_on_sample": round(float(np.mean(got == (gg_oracle.f64_from_bf16_bits(gg_oracle.bf16_bits_from_f64(ref["D"])) if bf16 else ref["W"]))), 5),
                               "max_err_over_S": float(np.max(err / np.maximum(ref["S"], 1e-300)))}
    print(json.dumps(out))


def bench_expert_mlp(args, cfg, dev):
    """Forward pass of the experts' MLP on the workload's routing: bf16 tokens [M_total, K] gathered by expert and
    quantised, GEMM with [G, N, K] (gate | up), silu(gate) * up + quantise, GEMM with [G, K, N/2] (down).  Padding-
    free: four kernels on M_total rows.  Padded (what a GEMM that needs 128-row groups forces on its neighbours):
    pad copy after the quantiser, both GEMMs and the activation on the padded rows, un-pad copy at the end."""
    import ctypes
    import numpy as np
    import torch

    import paper_2508_16584_amd as gg
    from workloads import group_sizes
    from workloads.quantize import quantize_b

    sizes = group_sizes(cfg, cfg.seed)
    G, M, K, N = cfg.G, int(np.sum(sizes)), cfg.K, cfg.N
    inter = N // 2
    km = args.sa_layout == "kmajor"
    sa_shape = (lambda rows, blocks: (blocks, rows)) if km else (lambda rows, blocks: (rows, blocks))
    gen = torch.Generator(device=dev)
    gen.manual_seed(cfg.seed)
    rng = np.random.default_rng(cfg.seed)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)).to(dev)
    X = torch.randn((M, K), generator=gen, device=dev, dtype=torch.float32).to(torch.bfloat16)
    src = torch.from_numpy(rng.permutation(M).astype(np.int32)).to(dev)
    B1 = torch.empty((G, N, K), dtype=torch.uint8, device=dev)
    SB1 = torch.empty((G, N // 128, K // 128), dtype=torch.float32, device=dev)
    B2 = torch.empty((G, K, inter), dtype=torch.uint8, device=dev)
    SB2 = torch.empty((G, K // 128, inter // 128), dtype=torch.float32, device=dev)
    for g in range(G):
        B1[g], SB1[g] = quantize_b(torch.randn((N, K), generator=gen, device=dev) * 0.02)
        B2[g], SB2[g] = quantize_b(torch.randn((K, inter), generator=gen, device=dev) * 0.02)
    cap = gg.padded_rows_cap(G, M)
    A1 = torch.empty((M, K), dtype=torch.uint8, device=dev)
    SA1 = torch.empty(sa_shape(M, K // 128), dtype=torch.float32, device=dev)
    H = torch.empty((M, N), dtype=torch.bfloat16, device=dev)
    A2 = torch.empty((M, inter), dtype=torch.uint8, device=dev)
    SA2 = torch.empty(sa_shape(M, inter // 128), dtype=torch.float32, device=dev)
    Y = torch.empty((M, K), dtype=torch.bfloat16, device=dev)
    H_pad = torch.empty((cap, N), dtype=torch.bfloat16, device=dev)
    A2_pad = torch.empty((cap, inter), dtype=torch.uint8, device=dev)
    SA2_pad = torch.empty(sa_shape(cap, inter // 128), dtype=torch.float32, device=dev)
    Y_pad = torch.empty((cap, K), dtype=torch.bfloat16, device=dev)

    def free_chain():
        gg.quantize_rows(X, src, A=A1, SA=SA1, sa_kmajor=km)
        gg.grouped_gemm(A1, SA1, B1, SB1, off, C=H, sa_kmajor=km)
        gg.swiglu_quantize_rows(H, A=A2, SA=SA2, sa_kmajor=km)
        gg.grouped_gemm(A2, SA2, B2, SB2, off, C=Y, sa_kmajor=km)

    def fused_chain():          # the activation and the second quantiser in the first GEMM's epilogue: three kernels
        gg.quantize_rows(X, src, A=A1, SA=SA1, sa_kmajor=km)
        gg.grouped_gemm_swiglu(A1, SA1, B1, SB1, off, A2=A2, SA2=SA2, sa_kmajor=km)
        gg.grouped_gemm(A2, SA2, B2, SB2, off, C=Y, sa_kmajor=km)

    def pad_chain():
        gg.quantize_rows(X, src, A=A1, SA=SA1, sa_kmajor=km)
        A_pad, SA_pad, poff = gg.pad(A1, SA1, off, sa_kmajor=km)
        gg.grouped_gemm_padded(A_pad, SA_pad, B1, SB1, poff, C_pad=H_pad, sa_kmajor=km)
        gg.swiglu_quantize_rows(H_pad, A=A2_pad, SA=SA2_pad, sa_kmajor=km)
        gg.grouped_gemm_padded(A2_pad, SA2_pad, B2, SB2, poff, C_pad=Y_pad, sa_kmajor=km)
        gg.unpad(Y_pad, off, poff, M, C=Y)

    def timed(fn):
        for _ in range(args.warmup):
            fn()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            fn()
        torch.cuda.synchronize()
        return (time.perf_counter() - t0) * 1e3 / args.steps

    n_ramp = clock_warmup(lambda i: free_chain(), args.clock_warmup_ms)
    t_free = timed(free_chain)
    y_free = Y.clone()
    t_fused, fused_same = None, None
    if inter % 128 == 0 and K % 256 == 0 and K >= 512 and 2 * inter * K < 2 ** 31:
        t_fused = timed(fused_chain)
        fused_same = bool(torch.equal(y_free.view(torch.int16), Y.view(torch.int16)))
    # the four-kernel padding-free chain recorded once into a HIP graph and replayed (the library only enqueues kernel
    # launches, so stream capture takes it as it is): what is left of the host's launch cost
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        free_chain()
    t_graph = timed(graph.replay)
    graph_same = bool(torch.equal(y_free.view(torch.int16), Y.view(torch.int16)))
    t_pad = timed(pad_chain)
    same = bool(torch.equal(y_free.view(torch.int16), Y.view(torch.int16)))
    flops = 2.0 * M * N * K + 2.0 * M * K * inter
    print(json.dumps({
        "metric": "expert MLP forward (quantise, GEMM, silu*up + quantise, GEMM), FP8 TFLOP/s of the two GEMMs on valid rows",
        "value": round(flops / (t_free * 1e-3) / 1e12, 2), "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(t_free, 4), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "bf16 tokens, fp8_e4m3 operands, fp32 accumulate, bf16 out", "data": "synthetic",
        "config": {"workload": args.workload + " routing", "op": "expert_mlp", "G": G, "M_total": M, "hidden": K,
                   "intermediate": inter, "sa_layout": "K-block-major" if km else "row-major",
                   "clock_warmup_launches": n_ramp},
        "graph_replay_ms": round(t_graph, 4), "graph_replay_output_bitwise_equal": graph_same,
        "fused_chain_ms": None if t_fused is None else round(t_fused, 4),
        "fused_chain_output_bitwise_equal": fused_same,
        "padded_chain_ms": round(t_pad, 4), "speedup_vs_padded_chain": round(t_pad / t_free, 4),
        "padded_chain_output_bitwise_equal": same,
        "note": "caches warm (same buffers every step); the padded chain adds a pad and an un-pad copy and runs the "
                "GEMMs and the activation on 128-row padded groups",
    }))


def bench_ceilings():
    """What this GPU sustains with the kernels' own instructions and nothing around them (include/gg_probe.h): one
    JSON line.  Each matrix loop runs for about 10 ms, long enough for the sustained clock."""
    import paper_2508_16584_amd as gg
    modes = ["16x16x128 accumulating", "16x16x128 from zero + 4 FMA (this algorithm's inner loop)",
             "32x32x64 accumulating", "2 x 32x32x64 per scale block + 16 FMA"]
    kinds = ["constant 1.0", "normal-like e4m3", "uniform random bytes"]
    mfma = {m: {k: round(gg.probe_mfma(mi, ki, 20000), 1) for ki, k in enumerate(kinds)} for mi, m in enumerate(modes)}
    mixes = [(0, 0, 0), (2, 0, 0), (4, 0, 0), (8, 0, 0), (0, 1, 0), (0, 2, 0), (0, 0, 1), (0, 0, 2), (2, 1, 1), (2, 1, 2)]
    issue = {f"+{a} scalar +{b} vector +{c} LDS reads per matrix instruction": round(gg.probe_issue_mix(a, b, c), 1) for a, b, c in mixes}
    hbm = {"read_GBps": round(gg.probe_hbm(0), 1), "copy_GBps": round(gg.probe_hbm(1), 1)}
    patterns = ["L2-resident contiguous 64 KB", "L2-resident column blocks [256 rows x 128 B] x 2",
                "kernel stream (4 x 8 tiles per die, K = 7168)"]
    fetch = {}
    for pi, pn in enumerate(patterns):
        fetch[pn] = {}
        for depth in (1, 2, 3, 4, 6):
            gbps, bpc = gg.probe_lds_fetch(pi, depth, 20)
            fetch[pn][f"depth {depth}"] = {"GBps": round(gbps, 1), "B_per_clk_per_CU_at_nominal_clock": round(bpc, 2)}
    print(json.dumps({"op": "ceilings", "mfma_fp8_TFLOPs": mfma,
                      "block_scaled_loop_on_constant_operands_with_more_instructions_TFLOPs": issue, "hbm": hbm, "l2_to_lds_fetch": fetch,
                      "peaks": {"mfma_fp8_dense_TFLOPs": 5000.0, "hbm_GBps": 8000.0}}))


def bench_kstep_parts():
    """The second GEMM kernel with parts of its K step left out (gg_probe_gemm_kstep), on two balanced problems of
    gate_up's N and K: 8 x 1152 rows in 192-row tiles and 8 x 1536 rows in 256-row tiles (768 tiles each: three full
    passes over 256 workgroups).  One JSON line; times are microseconds per launch, the ideal is the matrix pipe's
    time for the same tiles at the nominal clock.  Each build is launched once for every dispatch that is timed, so
    the same command under `rocprofv3 --pmc GRBM_GUI_ACTIVE` gives the cycles of every build."""
    import paper_2508_16584_amd as gg
    parts = [(0, "nothing left out (the kernel as launched)"), (4, "no barrier"), (8, "no LDS reads of activations and scales"),
             (16, "no waits for the fetches"), (20, "no waits for the fetches, no barrier"),
             (28, "no waits for the fetches, no barrier, no LDS reads (the fetched data moves beside the arithmetic, nothing waits for it)"),
             (92, "the same with the fetches landing in registers instead of LDS"),
             (32, "nothing left out, operands all zero bytes (same traffic, little power)"),
             (2, "fetches issued to nowhere (no traffic, zero operands)"), (1, "no fetches"), (5, "no fetches, no barrier"),
             (13, "no fetches, no barrier, no LDS reads (matrix instructions, FMAs, bookkeeping)")]
    out = {}
    for rows, per_group in ((192, 1152), (256, 1536)):
        res = {}
        for code, name in parts:
            res[name] = round(gg.probe_gemm_kstep(rows, code, 8, per_group, 4096, 7168, 20), 1)
        tiles_per_wg = 8 * (per_group // rows) * (4096 // 256) / 256.0
        ideal_cycles = tiles_per_wg * (7168 // 128) * (rows // 16) * 2 * 2 * 32   # per SIMD: 2 waves x (rows/16 x 2) instructions x 32 cycles
        out[f"{rows}x256 tiles, 8 groups x {per_group} rows, N=4096, K=7168"] = {
            "us_per_launch": res, "matrix_pipe_minimum_cycles": int(ideal_cycles),
            "matrix_pipe_minimum_us_at_2.4GHz": round(ideal_cycles / 2400.0, 1)}
    print(json.dumps({"op": "kstep_parts", "second_gemm_kernel_with_parts_of_its_k_step_left_out": out}))


def bench_wgrad_parts():
    """The narrow weight-gradient kernel (tiles of 256 x 128) with parts of a token block's work left out (gg_probe_wgrad_parts), on
    gate_up's layer, which itself takes the square tiles, with 8 equal groups of 1000 tokens (8 blocks each, the first and the last of them cut by a group boundary)
    and on a store-bound layer (32 groups of 48 tokens, same N and K).  One JSON line; microseconds per launch; the
    ideal is the matrix pipe's time for the same blocks at the nominal clock."""
    import paper_2508_16584_amd as gg
    parts = [(0, "nothing left out"), (2, "no stores"), (1, "no fetches"),
             (3, "neither (arithmetic, LDS reads, barrier, masks)"), (7, "the same without the barrier"),
             (11, "neither fetches nor stores, no byte masks"), (19, "neither fetches nor stores, no LDS reads"),
             (31, "matrix instructions and FMAs alone")]
    out = {}
    for groups, tokens in ((8, 1000), (32, 48)):
        res = {name: round(gg.probe_wgrad_parts(code, groups, tokens, 4096, 7168, 20), 1) for code, name in parts}
        first, last = [g * tokens // 128 for g in range(groups)], [(g * tokens + tokens - 1) // 128 for g in range(groups)]
        blocks = sum(b - a + 1 for a, b in zip(first, last))
        ideal_cycles = blocks * (4096 // 128) * (7168 // 256) * 128 * 32 / 1024.0     # 128 instructions per tile and block, 1024 SIMDs
        out[f"{groups} groups x {tokens} tokens, N=4096, K=7168"] = {
            "us_per_launch": res, "token_blocks_of_all_groups": blocks, "matrix_pipe_minimum_us_at_2.4GHz": round(ideal_cycles / 2400.0, 1),
            "dW_bytes": groups * 4096 * 7168 * 4}
    print(json.dumps({"op": "wgrad_parts", "weight_gradient_kernel_with_parts_left_out": out}))


def bench_pad_path(args, cfg, dev):
    """The comparison path of Sec. 3 step by step: pad (offsets + row copies), the GEMM on the padded problem, unpad.
    Each step is timed alone, `steps` launches back to back over rotating buffer sets (cold caches); the copies are
    HBM-bound: algorithmic bytes = what the step must read plus what it must write, each once."""
    import numpy as np
    import torch

    import paper_2508_16584_amd as gg
    from workloads import make_problem
    km = args.sa_layout == "kmajor"
    p = make_problem(cfg, device=dev)
    G, M, N, K = p["G"], p["M_total"], p["N"], p["K"]
    KB = K // 128
    cap = gg.padded_rows_cap(G, M)
    off = p["group_offsets"]
    SA = p["SA"].t().contiguous() if km else p["SA"]
    copies = args.copies or max(2, min(6, int(np.ceil(1.0e9 / (cap * (K + 2 * N))))))
    sets = []
    for i in range(copies):
        sets.append({
            "A": p["A"] if i == 0 else p["A"].clone(), "SA": SA if i == 0 else SA.clone(),
            "A_pad": torch.empty((cap, K), dtype=torch.uint8, device=dev),
            "SA_pad": torch.empty((KB, cap) if km else (cap, KB), dtype=torch.float32, device=dev),
            "C_pad": torch.empty((cap, N), dtype=torch.bfloat16, device=dev),
            "C": torch.empty((M, N), dtype=torch.bfloat16, device=dev)})
    poff = None
    for s_ in sets:      # every set holds a valid padded problem before anything is timed
        _, _, poff = gg.pad(s_["A"], s_["SA"], off, cap, sa_kmajor=km, A_pad=s_["A_pad"], SA_pad=s_["SA_pad"])
        gg.grouped_gemm_padded(s_["A_pad"], s_["SA_pad"], p["B"], p["SB"], poff, s_["C_pad"], sa_kmajor=km)
    torch.cuda.synchronize()
    m_pad = int(poff[-1].item())

    def pad_step(i):
        s_ = sets[i % copies]
        gg.pad(s_["A"], s_["SA"], off, cap, sa_kmajor=km, A_pad=s_["A_pad"], SA_pad=s_["SA_pad"])

    def gemm_step(i):
        s_ = sets[i % copies]
        gg.grouped_gemm_padded(s_["A_pad"], s_["SA_pad"], p["B"], p["SB"], poff, s_["C_pad"], sa_kmajor=km)

    def unpad_step(i):
        s_ = sets[i % copies]
        gg.unpad(s_["C_pad"], off, poff, M, C=s_["C"])

    row = K + 4 * KB
    steps_out = {}
    for name, fn, alg in (("pad", pad_step, M * row + m_pad * row + 8 * (G + 1)),
                          ("padded_gemm", gemm_step, None),
                          ("unpad", unpad_step, 2 * M * 2 * N)):
        clock_warmup(fn, args.clock_warmup_ms / 3)
        for i in range(args.warmup):
            fn(i)
        torch.cuda.synchronize()
        wall_ms, ev_ms = timed_region(fn, args.steps)
        entry = {"ms_per_step": round(wall_ms, 4), "kernel_avg_ms": round(ev_ms, 4)}
        if alg is not None:
            ach = alg / (ev_ms * 1e-3) / 1e9
            entry["roofline"] = {"bound": "hbm", "achieved": round(ach, 1), "peak": 8000.0, "unit": "GB/s",
                                 "frac": round(ach / 8000.0, 4), "algorithmic_bytes": int(alg), "traffic": None}
        else:
            entry["TFLOPs_on_valid_rows"] = round(2.0 * M * N * K / (wall_ms * 1e-3) / 1e12, 1)
            entry["variant"] = gg.variant_name(gg.auto_variant_padded(G, cap, N, K))
        steps_out[name] = entry
    total = sum(v["ms_per_step"] for v in steps_out.values())
    print(json.dumps({
        "metric": "pad-then-GEMM comparison path (Sec. 3), each step timed alone", "value": round(total, 4), "unit": "ms",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(total, 4), "higher_is_better": False,
        "scaling": "weak", "vs_baseline": None, "dtype": "u8 / fp32 / bf16 copies; fp8 e4m3 x e4m3 -> fp32 -> bf16 GEMM",
        "data": "synthetic",
        "config": {"workload": args.workload, "op": "pad_path", "G": G, "M_total": M, "M_pad": m_pad, "M_pad_cap": cap,
                   "N": N, "K": K, "sa_layout": args.sa_layout, "buffer_sets_rotated": copies},
        "pad": steps_out["pad"], "padded_gemm": steps_out["padded_gemm"], "unpad": steps_out["unpad"],
        "note": "pad = gg_pad_offsets_kernel + gg_pad_rows_kernel (reads the valid rows of A and S_A, writes the M_pad rows "
                "of the padded problem); unpad reads and writes the valid rows of the output",
    }))


def pmc_summary(folder):
    """Per kernel and counter, the mean over the dispatches in rocprofv3's `*counter_collection.csv` files under
    `folder` (one row per dispatch and counter), as a markdown table: what the summaries under profiles/ are made of."""
    import csv
    import glob
    acc = {}
    for path in sorted(glob.glob(os.path.join(folder, "**", "*counter_collection.csv"), recursive=True)):
        with open(path, newline="") as f:
            for row in csv.DictReader(f):
                key = (row["Kernel_Name"], row["Counter_Name"])
                acc.setdefault(key, []).append(float(row["Counter_Value"]))
                # the dispatch's duration as the profiler saw it (longer than an unprofiled launch)
                dur = (row["Kernel_Name"], "dispatch duration under the profiler, us (" + row["Counter_Name"] + " run)")
                acc.setdefault(dur, []).append((int(row["End_Timestamp"]) - int(row["Start_Timestamp"])) / 1e3)
    print("| kernel | counter | dispatches | mean | min | max |")
    print("|---|---|---|---|---|---|")
    for (kernel, counter), v in sorted(acc.items()):
        print(f"| `{kernel[:110]}` | {counter} | {len(v)} | {sum(v) / len(v):.1f} | {min(v):.1f} | {max(v):.1f} |")


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--wgrad-out", default="fp32", choices=["fp32", "bf16"], help="--op wgrad: the type of dW")
    ap.add_argument("--steps", type=int, default=60)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default="gate_up")
    ap.add_argument("--op", default="grouped_gemm", choices=["grouped_gemm", "quantize_rows", "swiglu_quantize_rows", "quantize_cols", "expert_mlp", "ceilings", "pad_path", "kstep_parts", "wgrad", "wgrad_parts"],
                    help="grouped_gemm: the hot path (default, the headline metric); quantize_rows: the producer of its "
                         "A operand on the same workload's activation shape; swiglu_quantize_rows: activation + quantiser "
                         "on the workload's output shape [M_total, N] (N = 2 x intermediate width); expert_mlp: the whole forward "
                         "chain quantise -> GEMM -> activation+quantise -> GEMM on the workload's routing, padding-free "
                         "against the same chain on 128-row padded groups; pad_path: the three steps of the pad-then-GEMM comparison path "
                         "(Sec. 3) each timed alone, the two copies against the HBM roofline; ceilings: no workload, the probes of "
                         "include/gg_probe.h (register-only matrix loops, HBM streams, the L2 -> LDS fetch stream); kstep_parts: no workload, "
                         "the second GEMM kernel timed with parts of its K step left out (fetches, barrier, LDS reads); wgrad: the variable-K "
                         "grouped GEMM of training (weight gradient) on the workload's layer")
    ap.add_argument("--clock-warmup-ms", type=float, default=150.0,
                    help="untimed launches for about this long before the W warm-up steps, so that the timed steps run at "
                         "the GPU's sustained clock (0: none)")
    ap.add_argument("--variant", type=int, default=-1)
    ap.add_argument("--sa-layout", choices=["kmajor", "row"], default="row",
                    help="storage order of the activation scales: row = [M_total, K/128], what the problem statement's "
                         "call gg_fp8_grouped_gemm takes (the default and the headline); kmajor = [K/128, M_total] "
                         "(GG_SA_KMAJOR of the _ex entry points: a few per cent faster, timed beside the headline)")
    ap.add_argument("--copies", type=int, default=0, help="input copies to rotate over (0 = enough for 1 GB)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-pad-path", action="store_true")
    ap.add_argument("--no-other-layout", "--no-row-major-compare", dest="no_other_layout", action="store_true",
                    help="skip the second timed loop with the other storage order of the activation scales")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a plain 1 GiB device copy (for scaling rocprofv3 FETCH_SIZE / WRITE_SIZE)")
    ap.add_argument("--pmc-summary", metavar="DIR", default=None,
                    help="no GPU work: print per-kernel means of the counters in rocprofv3's counter_collection.csv files under DIR")
    args = ap.parse_args()
    if args.pmc_summary:
        pmc_summary(args.pmc_summary)
        return
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs on ONE GPU (groups shard by expert across GPUs with no exchange inside the "
              "GEMM; nothing here uses a second GPU). Run with --gpus 1.", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import paper_2508_16584_amd as gg
    from workloads import CONFIGS, make_problem

    gg.load_library()      # fails loudly if the HIP library has not been built
    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(2)
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    if args.op == "ceilings":
        bench_ceilings()
        return
    if args.op == "wgrad_parts":
        bench_wgrad_parts()
        return
    if args.op == "kstep_parts":
        bench_kstep_parts()
        return
    cfg = CONFIGS[args.workload]
    if args.op == "wgrad":
        bench_wgrad(args, cfg, dev)
        return
    if args.op in ("quantize_rows", "swiglu_quantize_rows", "quantize_cols"):
        bench_quantize_rows(args, cfg, dev)
        return
    if args.op == "expert_mlp":
        bench_expert_mlp(args, cfg, dev)
        return
    if args.op == "pad_path":
        bench_pad_path(args, cfg, dev)
        return
    p = make_problem(cfg, device=dev)
    G, M, N, K = p["G"], p["M_total"], p["N"], p["K"]
    sizes = p["sizes"]
    flops = 2.0 * M * N * K
    alg_bytes = algorithmic_bytes(sizes, N, K)

    km = args.sa_layout == "kmajor"
    # ---- input copies to rotate over (cold caches) ---------------------------------------------
    # The headline is the call of the problem statement, gg_fp8_grouped_gemm, whose activation scales are row-major
    # [M_total, K/128] (Table 1 / App. A); --sa-layout kmajor times gg_fp8_grouped_gemm_ex with GG_SA_KMAJOR instead.
    # Whichever is not the headline is timed in a second loop of the same shape and reported beside it.
    per_set = alg_bytes
    copies = args.copies or max(2, min(8, int(np.ceil(1.0e9 / per_set))))
    ws_bytes = gg.workspace_bytes(G, M, N, K)
    sets = []
    for i in range(copies):
        if i == 0:
            s = {k: p[k] for k in ("A", "SA", "B", "SB", "group_offsets")}
        else:
            s = {k: p[k].clone() for k in ("A", "SA", "B", "SB", "group_offsets")}
        s["SA_row"] = s.pop("SA")                          # [M_total, K/128]
        s["SA_km"] = s["SA_row"].t().contiguous()          # [K/128, M_total]
        s["C"] = torch.empty((M, N), dtype=torch.bfloat16, device=dev)
        sets.append(s)
    ws = torch.zeros(max(ws_bytes, 1), dtype=torch.uint8, device=dev)

    def make_step(kmajor):
        def step(i):
            s = sets[i % copies]
            gg.grouped_gemm(s["A"], s["SA_km" if kmajor else "SA_row"], s["B"], s["SB"],
                            s["group_offsets"], C=s["C"], variant=args.variant, sa_kmajor=kmajor, workspace=ws)
        return step

    step = make_step(km)
    torch.cuda.reset_peak_memory_stats()
    n_ramp = clock_warmup(step, args.clock_warmup_ms)
    for i in range(args.warmup):
        step(i)
    torch.cuda.synchronize()
    ms_per_step, kern_avg_ms = timed_region(step, args.steps)
    kern_ms = per_launch_ms(step, args.steps)

    if args.copy_calibration:
        copy_calibration(dev)

    # hot-cache number (same buffers every step), secondary
    for _ in range(3):
        step(0)
    torch.cuda.synchronize()
    h0, h1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    h0.record()
    for _ in range(20):
        step(0)
    h1.record()
    torch.cuda.synchronize()
    hot_ms = h0.elapsed_time(h1) / 20

    # the same launches with the other storage order of the activation scales
    other = None
    if not args.no_other_layout:
        step_o = make_step(not km)
        for i in range(args.warmup):
            step_o(i)
        o_ms, o_kern_ms = timed_region(step_o, args.steps)       # the same timed region as the headline's
        other = {"entry_point": "gg_fp8_grouped_gemm_ex + GG_SA_KMAJOR" if not km else "gg_fp8_grouped_gemm",
                 "value": round(flops / (o_ms * 1e-3) / 1e12, 2), "unit": "TFLOP/s", "ms_per_step": round(o_ms, 4),
                 "frac_of_fp8_mfma_peak": round(flops / (o_kern_ms * 1e-3) / 1e12 / FP8_MFMA_PEAK_TFLOPS, 4)}
        step(0)                                             # C of set 0 is the headline layout's again (bitwise the same)

    value = flops / (ms_per_step * 1e-3) / 1e12
    if cfg.bound == "hbm":
        achieved = alg_bytes / (kern_avg_ms * 1e-3) / 1e9
        roof = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": round(achieved / HBM_PEAK_GBS, 4)}
    else:
        achieved = flops / (kern_avg_ms * 1e-3) / 1e12
        roof = {"bound": "mfma", "achieved": round(achieved, 1), "peak": FP8_MFMA_PEAK_TFLOPS, "unit": "TFLOP/s",
                "frac": round(achieved / FP8_MFMA_PEAK_TFLOPS, 4)}
    used = args.variant if args.variant >= 0 else gg.auto_variant(p["G"], p["M_total"], p["N"], p["K"])
    vname = gg.variant_name(used)
    roof["traffic"] = profiled_traffic("grouped_gemm", args.workload, args.sa_layout, vname)
    roof["traffic_source"] = TRAFFIC_SOURCE if roof["traffic"] is not None else None
    # the kernel of the variant that the library expects for these sizes (gg_fp8_auto_variant), or of the one asked for
    name = {0: "gg_gemm_pc_kernel", 3: "gg_gemm_pc_kernel", 23: "gg_gemm_sm_kernel", 24: "gg_gemm_sm_kernel", 25: "gg_gemm_sm_kernel"}.get(
        used, "gg_gemm_rb_kernel" if "-rb" in vname and args.variant >= 0 else "gg_gemm_rb_any_kernel" if "-rb" in vname else "gg_gemm_kernel")
    on_device = args.variant < 0 and (used in (0, 3) or "-rb" in vname)       # these kernels settle the tile height themselves
    roof["kernel"] = f"{name} (height chosen on the device, expected: {vname})" if on_device else f"{name}<{vname}>"
    roof["kernel_avg_ms"] = round(kern_avg_ms, 4)
    roof["kernel_median_ms"] = round(float(np.median(kern_ms)), 4)
    roof["kernel_min_ms"] = round(float(kern_ms.min()), 4)
    roof["algorithmic_bytes"] = int(alg_bytes)
    roof["algorithmic_flops"] = flops

    out = {
        "metric": "FP8 TFLOPS on valid rows, padding-free block-scaled grouped GEMM",
        "value": round(value, 2), "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "fp8_e4m3 in, fp32 accumulate, bf16 out", "data": "synthetic",
        "config": {"workload": args.workload, "G": G, "M_total": M, "N": N, "K": K,
                   "group_sizes": cfg.sizes, "rows_min": int(sizes.min()), "rows_max": int(sizes.max()),
                   "input_copies_rotated": copies, "variant": gg.variant_name(args.variant) or "auto",
                   "clock_warmup_launches": n_ramp,
                   "entry_point": "gg_fp8_grouped_gemm_ex + GG_SA_KMAJOR" if km else
                                  ("gg_fp8_grouped_gemm" if args.variant < 0 else "gg_fp8_grouped_gemm_variant"),
                   "sa_layout": "K-block-major [K/128, M_total] (GG_SA_KMAJOR)" if km else "row-major [M_total, K/128]",
                   "workspace_bytes": int(ws_bytes)},
        "frac_of_fp8_mfma_peak": round(value / FP8_MFMA_PEAK_TFLOPS, 4),
        "hot_cache_ms": round(hot_ms, 4),
        "roofline": roof,
    }
    if other:
        out["sa_kmajor" if not km else "sa_row_major"] = other

    # ---- pad-then-GEMM comparison path (Sec. 3) -------------------------------------------------
    if not args.no_pad_path:
        cap = gg.padded_rows_cap(G, M)
        mem0 = torch.cuda.memory_allocated()
        A_pad = torch.empty((cap, K), dtype=torch.uint8, device=dev)
        SA_pad = torch.empty((K // 128, cap) if km else (cap, K // 128), dtype=torch.float32, device=dev)
        flags = 2 if km else 0                                   # GG_SA_KMAJOR
        poff = torch.empty(G + 1, dtype=torch.int32, device=dev)
        C_pad = torch.empty((cap, N), dtype=torch.bfloat16, device=dev)
        ws_pad = torch.zeros(max(gg.workspace_bytes(G, cap, N, K), 1), dtype=torch.uint8, device=dev)
        GG_PADDED_GROUPS = 4      # what gg_fp8_grouped_gemm_padded passes: every group is a multiple of 128 rows
        pad_alloc = torch.cuda.memory_allocated() - mem0 - ws_pad.numel()
        lib = gg.load_library()
        import ctypes
        vp = lambda t: ctypes.c_void_p(t.data_ptr())
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

        def pad_step(i, with_unpad):
            s = sets[i % copies]
            rc = lib.gg_fp8_pad_ex(vp(s["A"]), vp(s["SA_km" if km else "SA_row"]), vp(s["group_offsets"]), vp(A_pad), vp(SA_pad), vp(poff),
                                   G, M, cap, K, stream, flags)
            rc |= lib.gg_fp8_grouped_gemm_ex(vp(A_pad), vp(SA_pad), vp(s["B"]), vp(s["SB"]), vp(poff), vp(C_pad),
                                             G, cap, N, K, vp(ws_pad), ws_pad.numel(), stream, -1, flags | GG_PADDED_GROUPS)
            if with_unpad:
                rc |= lib.gg_fp8_unpad(vp(C_pad), vp(s["group_offsets"]), vp(poff), vp(s["C"]), G, M, N, stream)
            assert rc == 0

        # the two loops alternate twice and each keeps its faster pass: the first loop after the headline's tends to run
        # in another clock state than the second, which once made the path WITH the extra copy the faster of the two
        res = {}
        for rnd in range(2):
            for with_unpad in (False, True):
                for i in range(max(3, args.warmup // 2)):
                    pad_step(i, with_unpad)
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                for i in range(args.steps):
                    pad_step(i, with_unpad)
                torch.cuda.synchronize()
                t = (time.perf_counter() - t0) * 1e3 / args.steps
                res[with_unpad] = min(t, res.get(with_unpad, t))
        m_pad = int(poff[-1].item())
        KB = K // 128
        row_bytes = K + 4 * KB + 2 * N                      # A, SA and C bytes per row
        weights = int(p["B"].numel() + p["SB"].numel() * 4)
        out["pad_path"] = {
            "pad_gemm_ms": round(res[False], 4), "pad_gemm_unpad_ms": round(res[True], 4),
            "speedup_vs_pad_gemm": round(res[False] / ms_per_step, 4),
            "speedup_vs_pad_gemm_unpad": round(res[True] / ms_per_step, 4),
            "M_pad": m_pad, "pad_overhead_rows": round(m_pad / M - 1, 4),
            "mem_saving_row_tensors": round(1 - M / m_pad, 4),          # 1 - bytes(A,SA,C)/bytes(A_pad,SA_pad,C_pad)
            "peak_bytes_padding_free": int(M * row_bytes + weights),
            "peak_bytes_pad_path": int(M * (K + 4 * KB) + m_pad * row_bytes + weights),
            # what the pad path's own buffers took in this run (torch's allocator, capacity M_pad_cap rows), next to
            # the analytic figure for the same buffers
            "pad_buffers_allocated_bytes": int(pad_alloc), "pad_buffers_analytic_bytes": int(cap * row_bytes + 4 * (G + 1)),
            "padded_gemm_variant": gg.variant_name(gg.auto_variant_padded(G, cap, N, K)),
            "paper_context": "1.7%-20.4% speed-up, up to 23.8% memory reduction on H800 (abstract)",
        }
        del A_pad, SA_pad, C_pad

    # ---- CPU oracle on a bounded sample of the same workload -------------------------------------
    if not args.no_cpu_baseline:
        from oracle import gg_oracle
        off = p["group_offsets"].cpu().numpy()
        per_group = 2048 if cfg.G <= 32 else 64
        groups = np.arange(G) if G <= 32 else np.arange(0, G, G // 32)
        rows = np.concatenate([np.arange(off[g], min(off[g + 1], off[g] + per_group)) for g in groups]).astype(np.int64)
        grp = np.searchsorted(off, rows, side="right") - 1
        used = np.unique(grp)
        ridx = torch.from_numpy(rows).to(dev)
        A_s, SA_s = p["A"][ridx].cpu().numpy(), p["SA"][ridx].cpu().numpy()
        B_s = p["B"][torch.from_numpy(used).to(dev)].cpu().numpy()
        SB_s = p["SB"][torch.from_numpy(used).to(dev)].cpu().numpy()
        off_s = np.concatenate([[0], np.cumsum([(grp == g).sum() for g in used])])
        t0 = time.perf_counter()
        ref = gg_oracle.grouped_gemm(A_s, SA_s, B_s, SB_s, off_s)
        cpu_s = time.perf_counter() - t0
        got = sets[0]["C"][ridx].cpu().view(torch.int16).numpy().view(np.uint16)
        # the tolerance of the parity tests, asserted on this sample (the abs-sum S is a second, untimed oracle pass):
        # |gpu - D| <= max(ulp, ulp/2 + 2^-10 S) for every element
        S = gg_oracle.grouped_gemm(A_s, SA_s, B_s, SB_s, off_s, with_abs_sum=True)["S"]
        err = np.abs(gg_oracle.f64_from_bf16_bits(got) - ref["D"])
        ulp = gg_oracle.bf16_ulp(ref["D"])
        bound = np.maximum(ulp, 0.5 * ulp + 2.0 ** -10 * S)
        assert np.all(err <= bound), f"bench.py: {int(np.sum(err > bound))} sampled outputs outside the tolerance"
        threads = int(os.environ.get("OMP_NUM_THREADS", os.cpu_count() or 1))
        try:
            from threadpoolctl import threadpool_info
            nt = [d.get("num_threads") for d in threadpool_info() if d.get("user_api") == "blas"]
            if nt:
                threads = int(max(nt))
        except Exception:
            pass
        out["cpu_baseline"] = {
            "value": round(2.0 * len(rows) * N * K / cpu_s / 1e12, 5), "unit": "TFLOP/s", "cores": threads,
            "kind": "oracle",
            "sample": f"first {per_group} rows of {len(groups)} groups ({len(rows)} rows x N={N} x K={K}), "
                      f"NumPy float64 oracle, {cpu_s:.1f} s",
            "gpu_bits_equal_oracle_on_sample": round(float(np.mean(got == ref["C"])), 5),
            "tolerance_asserted": "|gpu - D| <= max(ulp_bf16(D), ulp_bf16(D)/2 + 2^-10 S) on every sampled output",
            # in ulps of D: large only where D is a cancelled sum far below its terms (those outputs are judged by
            # the 2^-10 S term); max_err_over_bound is the worst ratio of error to tolerance (<= 1 by the assertion)
            "max_err_ulp": round(float(np.max(err / ulp)), 3),
            "max_err_over_bound": round(float(np.max(err / bound)), 4),
            "max_err_ulp_where_D_exceeds_S_over_1024": round(float(np.max((err / ulp)[np.abs(ref["D"]) >= S / 1024.0])), 3),
            "outputs_that_needed_the_floor": int(np.sum(err > ulp)), "outputs_compared": int(err.size),
        }

    print(json.dumps(out))


if __name__ == "__main__":
    main()

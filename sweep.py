#!/usr/bin/env python3
"""The paper's parameter sweep (Sec. 3.1, App. C.1) on one MI355X: padding-free grouped GEMM against
pad-then-GEMM over N, K in {3072..8192}, G in {4, 8, 16, 32}, M in {8192..65536}, with group sizes drawn by the
paper's generator.  Inputs are seeded and synthetic; both paths run the library's own kernels (the pad path is
pad kernels + the same GEMM on 128-aligned offsets + optional unpad), so the comparison isolates padding.

    python sweep.py                      # full grid (576 points), JSON lines to stdout, summary to stderr
    python sweep.py --grid quick         # the 16 corner points
    python sweep.py --out sweep.jsonl --summary sweep.md
    python sweep.py --build-fit                      # another experiment: the automatic choice on random problems.  A library that
                                                     # takes the kernels it chooses between by number (no GPU, needs hipcc) ...
    python sweep.py --tiles 400 --out tiles.jsonl    # ... every kernel's time ...
    python sweep.py --fit tiles.jsonl                # ... the estimates' constants from such files (no GPU, needs scipy)

Per point: time per launch of the three paths (HIP events on the launch stream; same buffers every launch, so small
problems are served by the Infinity Cache in all three paths alike, unless --cold flushes the caches before every
timed launch), TFLOP/s on valid rows, speed-up, and
the memory the row tensors save (1 - M / M_pad, the quantity whose magnitude the paper's abstract quotes).
The summary lists ranges and the Pearson correlations the paper discusses in Sec. 3.2 (speed-up against N, K, M,
G, M/G; memory saving against M/G).
"""
import argparse
import ctypes
import json
import math
import sys
import time

import numpy as np

# ---- the automatic choice between the kernels: random problems, every kernel's time, the estimates' constants ----------------
# What the choice is made between: the second and the fourth kernel with the height they choose themselves (numbers that only the
# library built by --build-fit takes), 128 x 128, the small tiles.  Beside them, the heights that those two choose between.
RB, PC = 29, 30
CHOICES = {RB: "second kernel", PC: "fourth kernel", 2: "128x128", 23: "32x64", 24: "32x128", 25: "64x128", 26: "16x16/8k", 27: "16x32/4k", 28: "16x32/4ko"}
HEIGHTS = {RB: {12: 256, 15: 224, 14: 192, 16: 128}, PC: {31: 32, 32: 64, 33: 96, 34: 128, 35: 160}}
# rows and columns of a tile, KB of weights that a workgroup has on their way, workgroups per compute unit, waves that the K blocks
# are dealt to, as in csrc/gg_fp8.hip
SMALL_TILES = {23: (32, 64, 24, 4, 1), 24: (32, 128, 32, 3, 1), 25: (64, 128, 32, 2, 1), 26: (16, 16, 32, 1, 8), 27: (16, 32, 32, 2, 4), 28: (16, 32, 32, 3, 4)}
FUSED_TILES = {14: (192, 256, 72, 1, 1), 15: (224, 256, 72, 1, 1), 12: (256, 256, 72, 1, 1), 24: (32, 256, 96, 1, 1), 25: (64, 256, 64, 1, 1)}


def fit_library():
    import paper_2508_16584_amd as gg
    return gg.library_path().replace("libgg_fp8.so", "libgg_fp8_fit.so")


def build_fit_library():
    from paper_2508_16584_amd import binding
    flags, binding.HIPCC_FLAGS = binding.HIPCC_FLAGS, binding.HIPCC_FLAGS + ["-DGG_FIT_BUILD"]
    binding._hipcc(binding.library_path().replace("libgg_fp8.so", "csrc/gg_fp8.hip"), fit_library(), False)
    binding.HIPCC_FLAGS = flags


def random_problem(rng, fused, min_flop=0.0):
    """G 1 ... 256, M 1 ... 32768, N and K 256 ... 8192 (fused: I to 4096), spread over the logarithm, a quarter with an N and an
    eighth with a K that are no multiples of 128; group sizes from even to strongly skewed."""
    from workloads.configs import WorkloadConfig, group_sizes
    spread = lambda lo, hi, step=1: min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random() / step)) * step))
    while True:
        G, M, K = spread(1, 256), spread(1, 32768), spread(512 if fused else 256, 8192, 128)
        N = 2 * spread(256, 4096, 128) if fused else spread(256, 8192, 8 if rng.random() < 0.25 else 128)
        if not fused and rng.random() < 0.125:
            K = spread(256, 8192, 16)
        if G * N * K > 2e9 or not min_flop <= 2.0 * M * N * K <= 4e11:
            continue
        law = str(rng.choice(["dirichlet100", "dirichlet1", "dirichlet0.3", "poisson128"]))
        return G, M, N, K, law, group_sizes(WorkloadConfig("random", 0, G, K, N, M, law, "mfma"), int(rng.integers(1 << 30)))


def time_tiles(args):
    import os

    import torch
    import paper_2508_16584_amd as gg
    from paper_2508_16584_amd import binding
    if not args.fused:
        if not os.path.exists(fit_library()):
            sys.exit(f"{fit_library()} is missing: build it with `python sweep.py --build-fit`")
        binding._LIB_NAME = os.path.basename(fit_library())
        assert gg.num_variants() == RB
    dev, rng = torch.device("cuda:0"), np.random.default_rng(args.seed)
    sink = open(args.out, "w") if args.out else sys.stdout
    gen = torch.Generator(device=dev)
    gen.manual_seed(args.seed)
    tiles = list(FUSED_TILES) if args.fused else list(CHOICES) + [v for h in HEIGHTS.values() for v in h]
    # operand bytes: normal samples in units of a quarter of e4m3's range, as a block quantiser leaves them
    pool = torch.cat([(torch.randn(1 << 24, generator=gen, device=dev) * 112).clamp(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8) for _ in range(8)])

    def operand(*shape):
        t = torch.empty(shape, dtype=torch.uint8, device=dev)
        flat, at = t.view(-1), 0
        while at < flat.numel():
            start = int(rng.integers(1 << 20)) * 16
            n = min(flat.numel() - at, pool.numel() - start)
            flat[at:at + n] = pool[start:start + n]
            at += n
        return t

    def captured(launch, n):
        launch(0)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for i in range(n):
                launch(i)
        return graph

    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def replay_us(graph, n):
        e0.record()
        graph.replay()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / n * 1e3

    for point in range(args.tiles):
        G, M, N, K, law, sizes = random_problem(rng, args.fused, 1e9 * args.min_gflop)
        km, KB, NB = bool(rng.random() < 0.5), -(-K // 128), -(-N // 128)
        off = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)).to(dev)
        copies = max(1, min(6, int(5e8 / (G * N * K)) + 1))             # weights of several layers in turn, as a model has them
        launches = copies * max(2, min(8, int(40 / (copies * (5 + 2.0 * M * N * K / 2e9)))))
        data = []
        for _ in range(copies):
            data.append((operand(M, K), torch.rand((KB, M) if km else (M, KB), generator=gen, device=dev) + 0.5, operand(G, N, K),
                         torch.rand((G, NB, KB), generator=gen, device=dev) + 0.5, off))
        if args.fused:
            A2 = torch.empty((M, N // 2), dtype=torch.uint8, device=dev)
            SA2 = torch.empty((N // 256, M) if km else (M, N // 256), device=dev)
            call = lambda i, v: gg.grouped_gemm_swiglu(*data[i % copies], A2=A2, SA2=SA2, sa_kmajor=km, variant=v)
        else:
            C = torch.empty((M, N), dtype=torch.bfloat16, device=dev)
            call = lambda i, v: gg.grouped_gemm(*data[i % copies], C=C, sa_kmajor=km, variant=v)
        graphs, times = {}, {}
        for v in [-1] + tiles:
            try:
                graphs[v] = captured(lambda i: call(i, v), launches)
            except gg.GGError as e:
                assert e.status == 3 and v >= 0                         # the tile does not take this N or K
        # the kernels in turn, in another order every time: what ran before moves the clock by several per cent
        for _ in range(6):
            for v in rng.permutation(list(graphs)).tolist():
                times.setdefault(v, []).append(replay_us(graphs[v], launches))
        times = {v: round(float(np.median(t[1:])), 2) for v, t in times.items()}
        del graphs
        sink.write(json.dumps(dict(G=G, M=M, N=N, K=K, law=law, km=km, fused=args.fused, sizes=sizes.tolist(), us=times)) + "\n")
        sink.flush()
        if point % 50 == 49:
            print(f"[tiles] {point + 1} problems", file=sys.stderr, flush=True)
        del data
    if args.out:
        sink.close()
        choice_summary([args.out])


def read_tiles(paths):
    rows = [json.loads(line) for path in paths for line in open(path)]
    for r in rows:
        r["us"] = {int(v): t for v, t in r["us"].items()}
    return rows


def choice_summary(paths):
    loss = sorted(r["us"][-1] / min(r["us"][v] for v in r["us"] if v >= 0 and (r["fused"] or v in CHOICES)) for r in read_tiles(paths))
    mean = math.exp(sum(map(math.log, loss)) / len(loss))
    print(f"{len(loss)} problems: the automatic choice takes {mean:.3f} of the best tile's time (geometric mean), "
          f"median {loss[len(loss) // 2]:.3f}, 9 of 10 within {loss[9 * len(loss) // 10]:.3f}, worst {loss[-1]:.2f}", file=sys.stderr)


def fit_large(rows):
    """The estimates of the second kernel, the fourth one and the 128 x 128 tile (kRbTime, kPcTime, kNarrowTime and the steps beside
    them in csrc/gg_fp8.hip), fitted to every other problem and tried on the rest.  The first two are fitted together: besides
    their errors, what the problems of 25 us and more lose where the smaller estimate is the wrong one counts."""
    from scipy.optimize import minimize
    G, M, N, K = (np.array([r[x] for r in rows], float) for x in "GMNK")
    T = {v: np.array([r["us"].get(v, np.inf) for r in rows]) for v in CHOICES}
    best = np.min(list(T.values()), axis=0)
    half = np.arange(len(rows)) % 2 == 0
    groups, blocks = G * (1 - np.exp(-M / G)), np.ceil(K / 128)
    row_tiles = {bm: np.maximum(groups, M / bm + 0.5 * groups) for bm in (32, 64, 96, 128, 160, 192, 224, 256)}
    step_cost = {128: 1.036, 192: 1.332, 224: 1.5, 256: 1.647}           # rb_step_cost

    def rounds(bm, columns, first):
        f = row_tiles[bm] * np.ceil(N / columns) / 256 * np.array([[0.96], [0.98], [1], [1.02], [1.04]])
        part = f - np.floor(f)
        return np.mean(np.floor(f) + np.where(part > 0, first + (1 - first) * part, 0), axis=0)

    def launch(steps, tbs, start, ragged, store):
        steps, data = np.where(K % 128 > 0, ragged, 1) * steps, (groups * N * K + M * (K + 2 * N)) / (tbs * 1e6)
        return start + (steps ** 4 + data ** 4) ** 0.25 + store * 2e-6 * M * N

    def pc(x):
        extra, step, step32, first, *rest = x
        return launch(np.min([(blocks + extra) * (step + step32 * row_tiles[32] / row_tiles[bm]) * rounds(bm, 256, first)
                              for bm in (32, 64, 96, 128, 160)], axis=0), *rest)

    def rb(x):
        extra, step, odd, first, *rest = x
        steps = np.min([(blocks + extra) * step * step_cost[bm] * rounds(bm, 256, first) for bm in step_cost], axis=0)
        return launch(np.where(blocks % 2 > 0, odd, 1) * steps, *rest)

    def narrow(x):
        extra, step, first, *rest = x
        return launch((blocks + extra) * step * rounds(128, 128, first), *rest)

    def bounded(x, first):                                              # a partly filled round costs a full one at most
        x = np.abs(x)
        x[first] = min(x[first], 1.0)
        return x

    def smallest(f, x):
        for _ in range(8):
            x = minimize(f, x, method="Nelder-Mead", options=dict(maxiter=4000, maxfev=4000, adaptive=True)).x
        return x

    both, large = np.isfinite(T[RB]), np.isfinite(T[RB]) & (np.minimum(T[RB], T[PC]) > 25)
    near = {v: T[v] < 1.5 * best for v in (RB, PC)}

    def losses(x):
        p, b = np.log(pc(bounded(x[:8], 3))), np.log(rb(bounded(x[8:], 3)))
        lp, lb = np.log(T[PC]), np.log(np.where(both, T[RB], 1))
        share = 1 / (1 + np.exp(np.clip((b - p) / 0.03, -50, 50)))       # of the second kernel, a step that has been rounded off
        return p - lp, b - lb, share * lb + (1 - share) * lp - np.minimum(lb, lp)

    def loss(x):
        ep, eb, lost = losses(x)
        return np.mean(lost[half & large]) + 0.1 * (np.mean(np.abs(ep[half & near[PC]]) ** 1.5) + np.mean(np.abs(eb[half & near[RB]]) ** 1.5))

    x = smallest(loss, np.array([2.0, 0.6, 0.1, 0.9, 6.0, 5.5, 1.1, 0.02, 3.0, 0.9, 1.05, 0.9, 6.0, 5.5, 1.1, 0.02]))
    ep, eb, _ = losses(x)
    wrong = np.where((rb(bounded(x[8:], 3)) <= pc(bounded(x[:8], 3)))[~half & large], T[RB][~half & large], T[PC][~half & large])
    names = "first tbs start ragged store".split()
    print("fourth kernel  ", *(f"{n} {v:.3f}" for n, v in zip(["extra", "step", "per 32 rows"] + names, bounded(x[:8], 3))),
          f"mean error {np.mean(np.abs(ep[~half & near[PC]])):.3f}")
    print("second kernel  ", *(f"{n} {v:.3f}" for n, v in zip(["extra", "step", "odd"] + names, bounded(x[8:], 3))),
          f"mean error {np.mean(np.abs(eb[~half & near[RB]])):.3f}")
    print(f"the one with the smaller estimate / the better one: {np.exp(np.mean(np.log(wrong / np.minimum(T[RB], T[PC])[~half & large]))):.4f} "
          f"on {len(wrong)} problems of 25 us and more that played no part")
    some = half & np.isfinite(T[2]) & (T[2] > 12)
    x = bounded(smallest(lambda x: np.mean(np.abs(np.log(narrow(bounded(x, 2)) / T[2])[some]) ** 1.5), np.array([3.0, 0.6, 0.8, 6.0, 4.5, 1.1, 0.05])), 2)
    other = ~half & np.isfinite(T[2]) & (T[2] > 12)
    print("128 x 128      ", *(f"{n} {v:.3f}" for n, v in zip(["extra", "step"] + names, x)),
          f"mean error {np.mean(np.abs(np.log(narrow(x) / T[2])[other])):.3f}")


def fit_tile(rows, v, tile, fused):
    """Constants of one small tile or tile of the fused kernel: latency, work, extra K steps, and the start-up time of the fifth kernel's.
    Returns them, their mean error and on how many problems that is (the fifth kernel's: on the half that was not fitted)."""
    from scipy.optimize import minimize
    BM, BN, kb_in_flight, per_cu, waves = tile
    f, t = [], []
    for r in rows:
        if v not in r["us"]:
            continue
        G, M, N, K = r["G"], r["M"], r["N"], r["K"]
        groups = G * (1 - math.exp(-M / G))
        tiles = max(groups, M / BM + 0.5 * groups) * -(-N // BN)
        weights = groups * N * K
        d = weights / (min(tiles, 256 * per_cu) * kb_in_flight * 1024) * (1.6 if weights > 64e6 else 0.7)
        f.append((tiles, -(-K // (128 * waves)), (weights + M * (K + (0.5 if fused else 2) * N)) / 6.8e6, d))
        t.append(r["us"][v])
    tiles, kb, c, d = np.array(f).T
    t, chain = np.array(t), waves > 1                 # the fifth kernel has no term for the weights in flight

    def estimate(p):
        latency, work, extra, start = [*np.exp(p), 4.2][:4]
        a, b = np.maximum(tiles / (256 * per_cu), 1) * (kb + extra) * latency, tiles * (kb + extra) * work / 256
        return start + (a ** 4 + b ** 4 + c ** 4 + (0 if chain else d ** 4)) ** 0.25

    def off(p, some):
        return np.abs(np.log(estimate(p) / t))[some]
    fitted, other = (slice(0, None, 2), slice(1, None, 2)) if chain else (slice(None), slice(None))
    fits = [minimize(lambda p: np.mean(off(p, fitted) ** 1.5), np.log([s, s] + ([1, 3] if chain else [4])), method="Nelder-Mead",
                     options=dict(maxiter=6000, maxfev=6000)) for s in (0.3, 1.2)]
    best = min(fits, key=lambda x: x.fun).x
    return np.exp(best), np.mean(off(best, other)), len(t[other])


def fit_tiles(paths):
    """The constants of the choice (kTileTimes, kChainTimes and what fit_large fits; kFusedTimes)."""
    rows = read_tiles(paths)
    fused = rows[0]["fused"]
    choice_summary(paths)
    if not fused:
        fit_large(rows)
    for v, tile in (FUSED_TILES if fused else SMALL_TILES).items():
        best, error, problems = fit_tile(rows, v, tile, fused)
        print(f"{v:3d} {tile[0]}x{tile[1]}{' fused' if fused else ''} latency {best[0]:.3f} work {best[1]:.3f} extra {best[2]:.2f}  "
              + (f"start {best[3]:.2f}  " if len(best) > 3 else "") + f"mean error {error:.3f} on {problems} problems")


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--grid", choices=["full", "quick"], default="full")
    ap.add_argument("--Ns", type=str, default=None, help="comma-separated override of the N values")
    ap.add_argument("--Ks", type=str, default=None)
    ap.add_argument("--Gs", type=str, default=None)
    ap.add_argument("--Ms", type=str, default=None)
    ap.add_argument("--steps", type=int, default=8)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--variant", type=int, default=-1, help="tile variant for every GEMM launch (-1: automatic)")
    ap.add_argument("--cold", action="store_true",
                    help="overwrite a 1 GiB buffer before every timed launch, so that neither the L2s nor the 256 MB "
                         "Infinity Cache hold any input (default: same buffers every launch, caches warm)")
    ap.add_argument("--free-only", action="store_true",
                    help="time the padding-free path only (for comparing tile variants; the pad columns repeat its time)")
    ap.add_argument("--sa-layout", choices=["kmajor", "row"], default="kmajor",
                    help="storage order of the activation scales: [K/128, M] (GG_SA_KMAJOR, default) or [M, K/128]")
    ap.add_argument("--seed", type=int, default=20250816)
    ap.add_argument("--out", type=str, default=None, help="write the JSON lines here instead of stdout")
    ap.add_argument("--summary", type=str, default=None, help="write the summary (markdown) here as well as to stderr")
    ap.add_argument("--tiles", type=int, default=0, help="time every tile on this many random problems instead of the grid")
    ap.add_argument("--min-gflop", type=float, default=0.0, help="with --tiles: larger problems only")
    ap.add_argument("--fused", action="store_true", help="with --tiles: the GEMM with the activation epilogue")
    ap.add_argument("--build-fit", action="store_true", help="compile the library that --tiles times (no GPU)")
    ap.add_argument("--fit", type=str, nargs="+", help="fit the constants of the choice to files that --tiles wrote")
    args = ap.parse_args()
    if args.build_fit:
        return build_fit_library()
    if args.tiles or args.fit:
        return fit_tiles(args.fit) if args.fit else time_tiles(args)

    import torch
    import paper_2508_16584_amd as gg
    from workloads.configs import paper_group_sizes
    from workloads.quantize import quantize_a, quantize_b

    if not torch.cuda.is_available():
        sys.exit("sweep.py needs an MI355X: no GPU visible")
    dev = torch.device("cuda:0")
    lib = gg.load_library()

    full = [3072, 4096, 5120, 6144, 7168, 8192]
    if args.grid == "full":
        Ns, Ks, Gs, Ms = full, full, [4, 8, 16, 32], [8192, 16384, 32768, 65536]
    else:
        Ns, Ks, Gs, Ms = [3072, 8192], [3072, 8192], [4, 32], [8192, 65536]
    pick = lambda s, d: [int(x) for x in s.split(",")] if s else d
    Ns, Ks, Gs, Ms = pick(args.Ns, Ns), pick(args.Ks, Ks), pick(args.Gs, Gs), pick(args.Ms, Ms)
    Gmax, Mmax = max(Gs), max(Ms)

    flags = 2 if args.sa_layout == "kmajor" else 0        # GG_SA_KMAJOR
    vp = lambda t: ctypes.c_void_p(t.data_ptr())
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    # bring the GPU to its sustained clock before the first grid point (about 150 ms of matrix work)
    wu = torch.randn((4096, 4096), device=dev, dtype=torch.bfloat16)
    t_wu = time.perf_counter()
    while time.perf_counter() - t_wu < 0.15:
        for _ in range(10):
            wu @ wu
        torch.cuda.synchronize()
    del wu
    sink = open(args.out, "w") if args.out else sys.stdout
    rows_out = []
    t_start = time.perf_counter()

    flush = torch.empty(1 << 30, dtype=torch.uint8, device=dev) if args.cold else None

    def timed(fn):
        for _ in range(args.warmup):
            fn()
        if flush is None:
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(args.steps):
                fn()
            e1.record()
            torch.cuda.synchronize()
            return e0.elapsed_time(e1) / args.steps        # ms per launch
        ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
        for e0, e1 in ev:
            flush.fill_(1)
            e0.record()
            fn()
            e1.record()
        torch.cuda.synchronize()
        return float(np.mean([e0.elapsed_time(e1) for e0, e1 in ev]))

    point = 0
    for K in Ks:
        gen = torch.Generator(device=dev)
        gen.manual_seed(args.seed + K)
        # activations for the largest M of the grid (any prefix of i.i.d. rows is a valid smaller problem)
        A = torch.empty((Mmax, K), dtype=torch.uint8, device=dev)
        SA = torch.empty((Mmax, K // 128), dtype=torch.float32, device=dev)
        for r0 in range(0, Mmax, 8192):
            rows = min(8192, Mmax - r0)
            x = torch.randn((rows, K), generator=gen, device=dev, dtype=torch.float32)
            A[r0:r0 + rows], SA[r0:r0 + rows] = quantize_a(x)
        for N in Ns:
            B = torch.empty((Gmax, N, K), dtype=torch.uint8, device=dev)
            SB = torch.empty((Gmax, N // 128, K // 128), dtype=torch.float32, device=dev)
            for g in range(Gmax):
                w = torch.randn((N, K), generator=gen, device=dev, dtype=torch.float32) * 0.02
                B[g], SB[g] = quantize_b(w)
            C = torch.empty((Mmax, N), dtype=torch.bfloat16, device=dev)
            ws = torch.zeros(max(gg.workspace_bytes(Gmax, Mmax, N, K), 4), dtype=torch.uint8, device=dev)
            cap_max = gg.padded_rows_cap(Gmax, Mmax)
            A_pad = torch.empty((cap_max, K), dtype=torch.uint8, device=dev)
            SA_pad = torch.empty((cap_max, K // 128), dtype=torch.float32, device=dev)
            C_pad = torch.empty((cap_max, N), dtype=torch.bfloat16, device=dev)
            for G in Gs:
                for M in Ms:
                    rng = np.random.default_rng([args.seed, N, K, G, M])
                    sizes = paper_group_sizes(M, G, rng)
                    off_h = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
                    off = torch.from_numpy(off_h).to(dev)
                    poff = torch.empty(G + 1, dtype=torch.int32, device=dev)
                    cap = gg.padded_rows_cap(G, M)
                    # the scales of the first M rows in the chosen order (SA_pad is written in the same order)
                    SA_M = SA[:M].t().contiguous() if flags else SA

                    def free_step():
                        rc = lib.gg_fp8_grouped_gemm_ex(vp(A), vp(SA_M), vp(B), vp(SB), vp(off), vp(C), G, M, N, K,
                                                        vp(ws), ws.numel(), stream, args.variant, flags)
                        assert rc == 0, gg.status_str(rc)

                    def pad_step(with_unpad):
                        rc = lib.gg_fp8_pad_ex(vp(A), vp(SA_M), vp(off), vp(A_pad), vp(SA_pad), vp(poff), G, M, cap, K, stream, flags)
                        rc |= lib.gg_fp8_grouped_gemm_ex(vp(A_pad), vp(SA_pad), vp(B), vp(SB), vp(poff), vp(C_pad),
                                                         G, cap, N, K, vp(ws), ws.numel(), stream, args.variant,
                                                         flags | (4 if args.variant < 0 else 0))      # GG_PADDED_GROUPS
                        if with_unpad:
                            rc |= lib.gg_fp8_unpad(vp(C_pad), vp(off), vp(poff), vp(C), G, M, N, stream)
                        assert rc == 0

                    t_free = timed(free_step)
                    m_pad = int(np.sum(128 * ((sizes + 127) // 128)))
                    if args.free_only:
                        t_pad = t_pad_unpad = t_free
                    else:
                        t_pad = timed(lambda: pad_step(False))
                        t_pad_unpad = timed(lambda: pad_step(True))
                        assert m_pad == int(poff[-1].item())
                    used = args.variant if args.variant >= 0 else gg.auto_variant(G, M, N, K)
                    rec = {
                        "N": N, "K": K, "G": G, "M": M, "M_pad": m_pad,
                        "rows_min": int(sizes.min()), "rows_max": int(sizes.max()),
                        "variant": gg.variant_name(used),
                        "t_free_us": round(t_free * 1e3, 2), "t_pad_gemm_us": round(t_pad * 1e3, 2),
                        "t_pad_gemm_unpad_us": round(t_pad_unpad * 1e3, 2),
                        "tflops": round(2.0 * M * N * K / (t_free * 1e-3) / 1e12, 1),
                        "speedup_vs_pad_gemm": round(t_pad / t_free, 4),
                        "speedup_vs_pad_gemm_unpad": round(t_pad_unpad / t_free, 4),
                        "mem_saving_row_tensors": round(1.0 - M / m_pad, 4),
                    }
                    rows_out.append(rec)
                    sink.write(json.dumps(rec) + "\n")
                    sink.flush()
                    point += 1
                    if point % 16 == 0:
                        print(f"[sweep] {point} points, {time.perf_counter() - t_start:.0f} s", file=sys.stderr, flush=True)
            del B, SB, C, A_pad, SA_pad, C_pad
        del A, SA
        torch.cuda.empty_cache()

    # ---- summary -----------------------------------------------------------------------------------------
    def col(name):
        return np.array([r[name] for r in rows_out], dtype=np.float64)

    def corr(x, y):
        return float(np.corrcoef(x, y)[0, 1]) if len(x) > 2 and np.std(x) > 0 and np.std(y) > 0 else float("nan")

    sp, spu, mem, tf = col("speedup_vs_pad_gemm"), col("speedup_vs_pad_gemm_unpad"), col("mem_saving_row_tensors"), col("tflops")
    Nc, Kc, Gc, Mc = col("N"), col("K"), col("G"), col("M")
    lines = [
        f"points: {len(rows_out)}  (N in {Ns}, K in {Ks}, G in {Gs}, M in {Ms}; variant {'auto' if args.variant < 0 else args.variant}; "
        f"activation scales {'K-block-major' if flags else 'row-major'}; caches {'flushed before every launch' if args.cold else 'warm'})",
        f"TFLOP/s on valid rows: min {tf.min():.0f}  median {np.median(tf):.0f}  max {tf.max():.0f}",
        f"speed-up over pad+GEMM: min {sp.min():.3f}  median {np.median(sp):.3f}  max {sp.max():.3f}",
        f"speed-up over pad+GEMM+unpad: min {spu.min():.3f}  median {np.median(spu):.3f}  max {spu.max():.3f}",
        f"memory saved on the row tensors (1 - M/M_pad): min {mem.min():.3f}  median {np.median(mem):.3f}  max {mem.max():.3f}",
        "Pearson r of the speed-up over pad+GEMM with N: %.3f, K: %.3f, M: %.3f, G: %.3f, M/G: %.3f" % (
            corr(Nc, sp), corr(Kc, sp), corr(Mc, sp), corr(Gc, sp), corr(Mc / Gc, sp)),
        "Pearson r of the memory saving with M: %.3f, G: %.3f, M/G: %.3f" % (corr(Mc, mem), corr(Gc, mem), corr(Mc / Gc, mem)),
    ]
    for G in Gs:
        for M in Ms:
            sel = (Gc == G) & (Mc == M)
            if sel.any():
                lines.append(f"G={G:2d} M={M:5d}: speed-up {sp[sel].mean():.3f} (with unpad {spu[sel].mean():.3f}), "
                             f"memory saved {mem[sel].mean():.3f}, TFLOP/s {tf[sel].mean():.0f}")
    text = "\n".join(lines)
    print(text, file=sys.stderr)
    if args.summary:
        with open(args.summary, "w") as f:
            f.write(text + "\n")
    if args.out:
        sink.close()


if __name__ == "__main__":
    main()

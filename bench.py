#!/usr/bin/env python3
"""Benchmark of the rotation-aware W4A4 linear layer on one MI355X.

A "step" is one pass of the whole hot path -- rotate + split + quantize (kernel A) and
the mixed-precision GEMM (kernel B), i.e. one dirotq_linear call -- over each of the four
FLUX.1-dev-shaped linears (M = 4608 tokens: fused QKV,
attention out-projection, fc1, fc2), on seeded synthetic outlier activations that are
resident in HBM before the timed region.  value = effective TOPS = sum(2 M N K) / time,
the dense layers the path replaces.  Prints ONE JSON line.
"""
from __future__ import annotations

import argparse
import dataclasses
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0      # MI355X dense bf16 MFMA
PEAK_FP8_TOPS = 5000.0         # MI355X dense fp8 MFMA (int8 has the same peak)
PEAK_FP6_TOPS = 10000.0        # MI355X dense FP6 MFMA: the codes of the pipelined and the 128 x 128 tiled kernels run on it;
                               # fractions of kernel B keep the fp8 peak in every workload, so that they compare
PEAK_HBM_GBS = 8000.0


def log(msg: str) -> None:
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def algorithmic(shape):
    """Algorithmic flops/ops and HBM bytes per launch of each kernel (what the method
    itself must compute and move, every operand once)."""
    M, K, N, r, g = shape.M, shape.K, shape.N, shape.r, shape.g
    G = (K - r) // g
    inter = 2 * M * r + M * (K - r) // 2 + 2 * M * G            # x_h + packed x_l + s_x
    blob = 2 * N * r + N * (K - r) // 2 + 2 * N * G
    return {
        "A_flops": 2.0 * M * K * K,
        "A_bytes": 2 * M * K + 2 * K * K + inter,
        "B_ops": 2.0 * M * N * (K - r) + 2.0 * M * N * r,
        "B_code_ops": 2.0 * M * N * (K - r),
        "B_bytes": inter + blob + 2 * M * N,
        "layer_ops": 2.0 * M * N * K,
        "gemm_bytes": 2 * M * K + 2 * N * K + 2 * M * N,
    }


def bench_w4a16(args, shapes, B, I, np, torch) -> int:
    """The W4A16 GEMM on every layer shape of the workload (weights quantized without rotation
    by dirotq_prepare_weights with Q = I), against the bf16 GEMM of the same shape."""
    dev = "cuda"
    layers = []
    for shp in shapes:
        L = I.make_layer(shp)
        W = torch.from_numpy(L.W).to(dev)
        blob = B.prepare_weights(W, torch.eye(shp.K, dtype=torch.float32, device=dev), 0, shp.g)
        if args.tokens:
            shp = dataclasses.replace(shp, M=min(args.tokens, shp.M))
        x = torch.from_numpy(np.ascontiguousarray(L.x_bits[:shp.M]).view(np.int16)).to(dev).view(torch.bfloat16)
        layers.append(dict(shape=shp, x=x, blob=blob, Wb=W.to(torch.bfloat16),
                           y=torch.empty((shp.M, shp.N), dtype=torch.bfloat16, device=dev)))
        del W
        torch.cuda.synchronize()
        log(f"inputs for {shp.name} ready")

    def step():
        for Ld in layers:
            s = Ld["shape"]
            B.w4a16_gemm(Ld["x"], Ld["blob"], s.N, s.g, out=Ld["y"])

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(args.steps):
        step()
    e1.record()
    torch.cuda.synchronize()
    ms_per_step = e0.elapsed_time(e1) / args.steps
    total_ops = sum(2.0 * Ld["shape"].M * Ld["shape"].N * Ld["shape"].K for Ld in layers)
    value = total_ops / (ms_per_step * 1e-3) / 1e12
    per_layer, sum_ms, bf16_ms = [], 0.0, 0.0
    for Ld in layers:
        s = Ld["shape"]
        ts, tg = [], []
        yb = torch.empty_like(Ld["y"])
        for fn, acc in ((lambda: B.w4a16_gemm(Ld["x"], Ld["blob"], s.N, s.g, out=Ld["y"]), ts),
                        (lambda: torch.matmul(Ld["x"], Ld["Wb"].t(), out=yb), tg)):
            fn()
            torch.cuda.synchronize()
            for _ in range(max(5, args.steps)):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                fn()
                b.record()
                torch.cuda.synchronize()
                acc.append(a.elapsed_time(b))
        t, g_ms = float(np.mean(ts)), float(np.mean(tg))
        rel = float((Ld["y"].float() - yb.float()).norm() / yb.float().norm())
        sum_ms += t
        bf16_ms += g_ms
        wbytes = s.N * s.K // 2 + 2 * s.N * (s.K // s.g)
        per_layer.append({"layer": s.name, "M": s.M, "K": s.K, "N": s.N, "g": s.g, "w4a16_gemm_ms": round(t, 4),
                          "bf16_gemm_ms": round(g_ms, 4), "frac_bf16_peak": round(2.0 * s.M * s.N * s.K / (t * 1e-3) / 1e12 / PEAK_BF16_TFLOPS, 4),
                          "weight_bytes_vs_bf16": round(wbytes / (2.0 * s.N * s.K), 4), "rel_err_vs_bf16_gemm": round(rel, 5)})
        log(f"{s.name}: w4a16 {t:.3f} ms  bf16 GEMM {g_ms:.3f} ms")
    ach = total_ops / (sum_ms * 1e-3) / 1e12
    roof = {"kernel": "w4a16_gemm_kernel", "bound": "mfma", "dtype": "bf16", "achieved": round(ach, 3),
            "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s", "frac": round(ach / PEAK_BF16_TFLOPS, 5),
            "avg_launch_ms": round(sum_ms / len(layers), 5), "traffic": None}
    if 0 < args.tokens <= 32:
        # every operand once: packed codes + scales + activations + output
        nbytes = sum(Ld["shape"].N * Ld["shape"].K // 2 + 2 * Ld["shape"].N * (Ld["shape"].K // Ld["shape"].g) +
                     2 * Ld["shape"].M * (Ld["shape"].K + Ld["shape"].N) for Ld in layers)
        gbs = nbytes / (sum_ms * 1e-3) / 1e9
        roof = {"kernel": "w4a16_eight_kernel" if args.tokens <= 8 else "w4a16_few_kernel", "bound": "hbm", "achieved": round(gbs, 1), "peak": 8000.0, "unit": "GB/s",
                "frac": round(gbs / 8000.0, 5), "avg_launch_ms": round(sum_ms / len(layers), 5),
                "algorithmic_bytes_per_launch": nbytes / len(layers), "traffic": None}
    out = {"metric": "effective TOPS of the W4A16 linear (16-bit activations, 4-bit per-group weights)",
           "value": round(value, 3), "unit": "TOPS", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
           "ms_per_step": round(ms_per_step, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
           "dtype": "bf16 (exact int4 codes as bf16, fp32 accumulate)", "data": "synthetic",
           "config": {"workload": f"{args.workload}-shaped layers through dirotq_w4a16_gemm, one call per layer per step",
                      "seed": 0},
           "speedup_vs_bf16_gemm": round(bf16_ms / ms_per_step, 4),
           "roofline": roof, "layers": per_layer, "cpu_baseline": None}
    print(json.dumps(out), flush=True)
    return 0


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--no-cpu-baseline", action="store_true", help="skip the oracle timing leg")
    ap.add_argument("--workload", default="flux", choices=["flux", "pixart", "small", "sweep", "ablation"],
                    help="flux = the benchmark; pixart = four PixArt-Sigma-shaped layers; small = M=256, K=N=1152; "
                         "sweep = token sweep on the PixArt fc1 shape; ablation = rank/group grid on the FLUX fc2 shape")
    ap.add_argument("--residual-rotation", action="store_true",
                    help="fold a random orthogonal rotation of the 4-bit subspace into Q (Q = [U_h, U_l R])")
    ap.add_argument("--shared-input", action="store_true",
                    help="flux only: fused QKV and fc1 read the same activations (as in FLUX's single-stream blocks): "
                         "one dirotq_linear_shared call rotates and quantizes them once for both GEMMs")
    ap.add_argument("--asym", action="store_true",
                    help="asymmetric activation quantizer (zero-point min, 16 unsigned levels): the *_asym entry points")
    ap.add_argument("--a8", action="store_true",
                    help="8-bit per-token activations against the same 4-bit weights: the *_a8 entry points")
    ap.add_argument("--w4a16", action="store_true",
                    help="time dirotq_w4a16_gemm (16-bit activations, 4-bit weights, no rotation) on the workload's "
                         "layer shapes instead of the W4A4 layer")
    ap.add_argument("--graph", action="store_true",
                    help="also record one step into a HIP graph and time its replays (graph_ms_per_step); the "
                         "headline value stays the eager one")
    ap.add_argument("--tokens", type=int, default=0,
                    help="with --w4a16: use only the first TOKENS tokens of each layer's activations (<= 32 takes "
                         "the few-token kernel, which is bound by the weight stream)")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also launch a plain elementwise copy of known size (256 MiB read + 256 MiB written), "
                         "the reference the FETCH_SIZE / WRITE_SIZE counters are scaled by")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build is single-GPU by design (one process, one MI355X, no collectives); "
              "run with --gpus 1", file=sys.stderr)
        return 2

    import numpy as np
    import torch

    from paper_2605_16732_amd import binding as B
    from paper_2605_16732_amd import inputs as I

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        return 3
    B.lib()                                           # fail loudly if the HIP library is not built
    torch.cuda.set_device(0)
    dev = "cuda"
    shapes = {"flux": I.FLUX, "pixart": I.PIXART, "small": [I.SMALL], "sweep": I.TOKEN_SWEEP,
              "ablation": I.ABLATION}[args.workload]

    def dev_bf16(bits):
        return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(dev).view(torch.bfloat16)

    if args.w4a16:
        return bench_w4a16(args, shapes, B, I, np, torch)

    # ---- inputs, resident in HBM before anything is timed ---------------------------
    layers = []
    t0 = time.time()
    shared = None                                     # ablation: one set of draws for every (r, g)
    for shp in shapes:
        if args.workload == "ablation":
            if shared is None:
                L = I.make_layer(I.FLUX[3], residual_rotation=args.residual_rotation)   # same draws as flux_fc2
                shared = (L, torch.from_numpy(L.Q32).to(dev), torch.from_numpy(L.W).to(dev))
                shared += (B.prepare_rotation(shared[1]), dev_bf16(L.x_bits), shared[2].to(torch.bfloat16))
            L, Q32, W, Qt, x, Wb = shared
            blob = B.prepare_weights(W, Q32, shp.r, shp.g)
        else:
            L = I.make_layer(shp, residual_rotation=args.residual_rotation)
            W = torch.from_numpy(L.W).to(dev)
            if args.shared_input and shp.name == "flux_fc1":
                # fc1 reads the QKV layer's activations through the QKV layer's rotation
                L0 = layers[0]["host"]
                Q32 = torch.from_numpy(L0.Q32).to(dev)
                Qt, x = layers[0]["Qt"], layers[0]["x"]
            else:
                Q32 = torch.from_numpy(L.Q32).to(dev)
                Qt = B.prepare_rotation(Q32)
                x = dev_bf16(L.x_bits)
            blob = B.prepare_weights(W, Q32, shp.r, shp.g)
            Wb = W.to(torch.bfloat16)                 # comparator: plain bf16 GEMM, same shape
            del Q32, W
        ws_bytes = B.a8_workspace_bytes(shp.M, shp.K, shp.r) if args.a8 else B.workspace_bytes(shp.M, shp.K, shp.r, shp.g)
        ws = torch.empty(ws_bytes, dtype=torch.uint8, device=dev)
        y = torch.empty((shp.M, shp.N), dtype=torch.bfloat16, device=dev)
        G = shp.G
        parts = (torch.empty((shp.M, shp.r), dtype=torch.bfloat16, device=dev),
                 torch.empty((shp.M, (shp.K - shp.r) // 2), dtype=torch.uint8, device=dev),
                 torch.empty((G, shp.M), dtype=torch.float16, device=dev))
        if args.asym:
            parts = parts + (torch.empty((G, shp.M), dtype=torch.float16, device=dev),)
        scratch = None
        if args.a8:
            parts = (parts[0], torch.empty((shp.M, shp.K - shp.r), dtype=torch.uint8, device=dev),
                     torch.empty((shp.M,), dtype=torch.float16, device=dev))
            scratch = torch.empty(B.a8_scratch_bytes(shp.M, shp.K, shp.r), dtype=torch.uint8, device=dev)
        layers.append(dict(shape=shp, x=x, Qt=Qt, blob=blob, ws=ws, y=y, Wb=Wb, parts=parts, host=L, scratch=scratch))
        torch.cuda.synchronize()
        log(f"inputs for {shp.name} ready ({time.time() - t0:.0f} s)")

    if args.calibrate_copy:
        ca = torch.ones(64 * 1024 * 1024, dtype=torch.float32, device=dev)
        cb = torch.empty_like(ca)
        for _ in range(3):
            torch.mul(ca, 1.0, out=cb)              # one elementwise kernel: reads 256 MiB, writes 256 MiB
        torch.cuda.synchronize()
        del ca, cb

    f_linear = B.linear_asym if args.asym else B.linear
    f_rq = B.rotate_quantize_asym if args.asym else B.rotate_quantize
    f_gemm = B.w4a4_gemm_asym if args.asym else B.w4a4_gemm

    if args.a8:
        if args.asym:
            print("bench.py: --a8 and --asym are different activation quantizers", file=sys.stderr)
            return 2
        f_linear, f_gemm = B.linear_a8, B.w4a8_gemm

    if args.shared_input and (args.workload != "flux" or args.asym or args.a8):
        print("bench.py: --shared-input applies to the symmetric flux workload", file=sys.stderr)
        return 2

    def step():
        for i, Ld in enumerate(layers):
            s = Ld["shape"]
            if args.shared_input and i == 0:
                L2 = layers[2]
                B.linear_shared(Ld["x"], Ld["Qt"], [Ld["blob"], L2["blob"]], [s.N, L2["shape"].N], s.r, s.g,
                                workspace=Ld["ws"], outs=[Ld["y"], L2["y"]])
            elif args.shared_input and i == 2:
                continue
            else:
                f_linear(Ld["x"], Ld["Qt"], Ld["blob"], s.N, s.r, s.g, workspace=Ld["ws"], out=Ld["y"])

    # ---- whole-step timing -----------------------------------------------------------
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t_wall = time.perf_counter()
    e0.record()
    for _ in range(args.steps):
        step()
    e1.record()
    torch.cuda.synchronize()
    wall_ms = (time.perf_counter() - t_wall) * 1e3
    ms_per_step = max(e0.elapsed_time(e1), 0.0) / args.steps
    ms_per_step = max(ms_per_step, 0.0)
    total_ops = sum(algorithmic(Ld["shape"])["layer_ops"] for Ld in layers)
    value = total_ops / (ms_per_step * 1e-3) / 1e12
    log(f"step {ms_per_step:.3f} ms (wall {wall_ms / args.steps:.3f} ms) -> {value:.1f} effective TOPS")

    graph_ms = None
    if args.graph:
        gr = torch.cuda.CUDAGraph()
        with torch.cuda.graph(gr):
            step()
        for _ in range(args.warmup):
            gr.replay()
        torch.cuda.synchronize()
        g0, g1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        g0.record()
        for _ in range(args.steps):
            gr.replay()
        g1.record()
        torch.cuda.synchronize()
        graph_ms = g0.elapsed_time(g1) / args.steps
        log(f"graph replay {graph_ms:.4f} ms per step (eager {ms_per_step:.4f} ms)")

    # ---- per-kernel timing (HIP events on the launch stream) ------------------------------
    # in-step: the step run as separate rotate_quantize / w4a4_gemm calls, layer after layer as in the timed
    # region, events around every kernel.  A step touches > 1 GB of operands (four blobs, four rotation
    # matrices, activations, outputs), far more than the 256 MB last-level cache, so every layer finds its
    # weights and its rotation cold, as in a model with hundreds of layers.  These durations feed `roofline`.
    # warm: the same launch repeated back to back (operands resident in the cache where they fit).
    reps = max(50, args.steps)

    def stats(ts):
        ts = sorted(ts)
        return {"mean": float(np.mean(ts)), "median": float(ts[len(ts) // 2]), "min": float(ts[0])}

    def fA(Ld):
        s = Ld["shape"]
        if args.a8:
            B.rotate_quantize_a8(Ld["x"], Ld["Qt"], s.r, out=Ld["parts"], scratch=Ld["scratch"])
        else:
            f_rq(Ld["x"], Ld["Qt"], s.r, s.g, out=Ld["parts"])

    def fB(Ld):
        s = Ld["shape"]
        f_gemm(*Ld["parts"], Ld["blob"], s.M, s.N, s.K, s.r, s.g, out=Ld["y"])

    def fL(Ld):
        s = Ld["shape"]
        f_linear(Ld["x"], Ld["Qt"], Ld["blob"], s.N, s.r, s.g, workspace=Ld["ws"], out=Ld["y"])

    def fG(Ld):
        torch.matmul(Ld["x"], Ld["Wb"].t(), out=Ld["yb"])

    for Ld in layers:
        Ld["yb"] = torch.empty_like(Ld["y"])
    kinds = (("A", fA), ("B", fB), ("L", fL), ("G", fG))
    ev = {k: [[] for _ in layers] for k, _ in kinds}
    def timed(k, fn, i, Ld, keep):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        fn(Ld)
        b.record()
        if keep:
            ev[k][i].append((a, b))

    for rep in range(reps + 2):
        for i, Ld in enumerate(layers):                      # the step, kernel by kernel: A B A B A B A B
            timed("A", fA, i, Ld, rep >= 2)
            timed("B", fB, i, Ld, rep >= 2)
        for i, Ld in enumerate(layers):                      # the step as the timed region runs it
            timed("L", fL, i, Ld, rep >= 2)
        for i, Ld in enumerate(layers):                      # the comparator
            timed("G", fG, i, Ld, rep >= 2)
    torch.cuda.synchronize()
    cold = {k: [stats([a.elapsed_time(b) for a, b in ev[k][i]]) for i in range(len(layers))] for k, _ in kinds}

    def time_warm(fn, Ld):
        fn(Ld)
        torch.cuda.synchronize()
        evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(reps)]
        for a, b in evs:
            a.record()
            fn(Ld)
            b.record()
        torch.cuda.synchronize()
        return stats([a.elapsed_time(b) for a, b in evs])

    per_layer = []
    for i, Ld in enumerate(layers):
        s = Ld["shape"]
        alg = algorithmic(s)
        tA, tB, tL, tG = cold["A"][i], cold["B"][i], cold["L"][i], cold["G"][i]
        wA, wB, wL, wG = (time_warm(fn, Ld) for _, fn in kinds)
        # error of the quantized layer against the bf16 GEMM of the same operands (fp32 math on the GPU)
        fL(Ld)
        dlt = (Ld["y"].float() - Ld["yb"].float())
        rel_err = float(dlt.norm() / Ld["yb"].float().norm())
        del dlt
        rnd = lambda d: {k: round(v, 4) for k, v in d.items()}
        # ideal-rate ceiling of the method on this shape: rotation (2 M K^2 at the bf16 rate) + 4-bit product
        # (at twice that rate) + 16-bit branch, against the bf16 GEMM of the layer at the same efficiency
        rho = s.r / s.K
        ceiling = 1.0 / (s.K / s.N + (1.0 - rho) / 2.0 + rho)
        per_layer.append({
            "layer": s.name, "M": s.M, "K": s.K, "N": s.N, "r": s.r, "g": s.g,
            "rotate_quantize_ms": round(tA["mean"], 4), "w4a4_gemm_ms": round(tB["mean"], 4),
            "linear_ms": round(tL["mean"], 4), "bf16_gemm_ms": round(tG["mean"], 4),
            "in_step_ms": {"rotate_quantize": rnd(tA), "w4a4_gemm": rnd(tB), "linear": rnd(tL), "bf16_gemm": rnd(tG)},
            "warm_ms": {"rotate_quantize": rnd(wA), "w4a4_gemm": rnd(wB), "linear": rnd(wL), "bf16_gemm": rnd(wG)},
            "rotate_quantize_frac_bf16_peak": round(alg["A_flops"] / (tA["mean"] * 1e-3) / 1e12 / PEAK_BF16_TFLOPS, 4),
            "w4a4_gemm_frac_fp8_peak": round(alg["B_code_ops"] / (tB["mean"] * 1e-3) / 1e12 / PEAK_FP8_TOPS, 4),
            "effective_tops": round(alg["layer_ops"] / (tL["mean"] * 1e-3) / 1e12, 2),
            "speedup_vs_bf16_gemm": round(tG["mean"] / tL["mean"], 4),
            "speedup_ceiling_at_ideal_rates": round(ceiling, 3),
            "hbm_gbs_algorithmic": round((alg["A_bytes"] + alg["B_bytes"]) / (tL["mean"] * 1e-3) / 1e9, 1),
            "rotate_quantize_share_of_layer": round(tA["mean"] / (tA["mean"] + tB["mean"]), 4),
            "rel_err_vs_bf16_gemm": round(rel_err, 5),
            "_tA": tA["mean"], "_tB": tB["mean"], "_mA": tA["median"], "_mB": tB["median"], "_alg": alg,
        })
        log(f"{s.name}: in-step A {tA['mean']:.3f} (median {tA['median']:.3f}, warm {wA['median']:.3f}) ms  "
            f"B {tB['mean']:.3f} (median {tB['median']:.3f}, warm {wB['median']:.3f}) ms  fused {tL['mean']:.3f} ms  "
            f"bf16 GEMM {tG['mean']:.3f} ms")

    # ---- measured matrix-pipe rates (MFMA-only loops), next to the datasheet peaks -------------
    measured_peaks = None
    probe_path = os.path.join(ROOT, "paper_2605_16732_amd", "libdirotq_probe.so")
    if os.path.exists(probe_path):
        import ctypes
        P = ctypes.CDLL(probe_path)
        P.dirotq_probe_mfma_rate.restype = ctypes.c_double
        P.dirotq_probe_mfma_rate.argtypes = [ctypes.c_int] * 3 + [ctypes.c_void_p] * 3
        blocks, iters = 256, 4000
        sink = torch.empty(blocks * 512, dtype=torch.float32, device=dev)
        measured_peaks = {}
        for data in ("random", "zeros"):
            seed = (torch.randint(0, 2 ** 31 - 1, (blocks * 512 * 8,), dtype=torch.int32, device=dev) if data == "random"
                    else torch.zeros(blocks * 512 * 8, dtype=torch.int32, device=dev))
            for kind, name in ((0, "bf16_32x32x16"), (1, "bf16_16x16x32"), (2, "fp8_32x32x64")):
                best = 0.0
                for _ in range(3):
                    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                    a.record()
                    fl = P.dirotq_probe_mfma_rate(kind, blocks, iters, seed.data_ptr(), sink.data_ptr(),
                                                  torch.cuda.current_stream().cuda_stream)
                    b.record()
                    torch.cuda.synchronize()
                    if fl > 0:
                        best = max(best, fl / (a.elapsed_time(b) * 1e-3) / 1e12)
                measured_peaks[f"{name}_{data}_operands_tflops"] = round(best, 1)
        log(f"measured MFMA-only rates: {measured_peaks}")

    # dominant kernel = the one with the larger summed duration over a step
    sumA = sum(p["_tA"] for p in per_layer)
    sumB = sum(p["_tB"] for p in per_layer)
    n_launch = len(per_layer)
    if sumA >= sumB:
        flops = sum(p["_alg"]["A_flops"] for p in per_layer)
        roofline = {"kernel": "rotate_quantize_kernel", "bound": "mfma", "dtype": "bf16",
                    "achieved": flops / (sumA * 1e-3) / 1e12, "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s",
                    "avg_launch_ms": sumA / n_launch, "launches_per_step": n_launch,
                    "algorithmic_flops_per_launch": flops / n_launch, "traffic": None}
    else:
        ops = sum(p["_alg"]["B_code_ops"] for p in per_layer)
        roofline = {"kernel": "w4a8_gemm_kernel" if args.a8 else "w4a4_gemm_kernel", "bound": "mfma", "dtype": "fp8",
                    "achieved": ops / (sumB * 1e-3) / 1e12, "peak": PEAK_FP8_TOPS, "unit": "TOP/s",
                    "avg_launch_ms": sumB / n_launch, "launches_per_step": n_launch,
                    "algorithmic_flops_per_launch": ops / n_launch, "traffic": None}
    roofline["frac"] = roofline["achieved"] / roofline["peak"]
    roofline["timing"] = (f"mean over {reps} in-step launches per layer shape (HIP events on the launch stream; operands cold: "
                          "a step cycles > 1 GB through the 256 MB last-level cache)")
    med = sum(p["_mA" if sumA >= sumB else "_mB"] for p in per_layer)
    roofline["frac_from_median"] = roofline["frac"] * (sumA if sumA >= sumB else sumB) / med
    if measured_peaks:
        mp = max(measured_peaks["bf16_32x32x16_random_operands_tflops"], measured_peaks["bf16_16x16x32_random_operands_tflops"]) \
            if sumA >= sumB else measured_peaks["fp8_32x32x64_random_operands_tflops"]
        roofline["measured_mfma_only_peak"] = mp
        roofline["frac_of_measured_peak"] = roofline["achieved"] / mp if mp > 0 else None
    # HBM traffic per launch from the committed rocprofv3 counter summary (FETCH_SIZE + WRITE_SIZE,
    # scaled by the copy-kernel calibration), if one exists for this kernel and workload
    tfile = os.path.join(ROOT, "profiles", f"{roofline['kernel']}_{args.workload}_hbm_traffic.txt")
    if os.path.exists(tfile):
        for line in open(tfile):
            if line.startswith("traffic_bytes_per_launch:"):
                roofline["traffic"] = float(line.split(":")[1])
        roofline["algorithmic_bytes_per_launch"] = sum(p["_alg"]["A_bytes" if sumA >= sumB else "B_bytes"]
                                                       for p in per_layer) / n_launch
    other = {"rotate_quantize_kernel": {"sum_ms_per_step": sumA,
                                        "frac_bf16_peak": sum(p["_alg"]["A_flops"] for p in per_layer) / (sumA * 1e-3) / 1e12 / PEAK_BF16_TFLOPS},
             "w4a4_gemm_kernel": {"sum_ms_per_step": sumB,
                                  "frac_fp8_peak": sum(p["_alg"]["B_code_ops"] for p in per_layer) / (sumB * 1e-3) / 1e12 / PEAK_FP8_TOPS}}
    bf16_ms = sum(p["bf16_gemm_ms"] for p in per_layer)
    for p in per_layer:
        for k in ("_tA", "_tB", "_mA", "_mB", "_alg"):
            p.pop(k)

    # ---- CPU baseline: the oracle as it stands, bounded sample --------------------------
    cpu = None
    if not args.no_cpu_baseline:
        from oracle import dirotq_oracle as O
        Ld = layers[min(2, len(layers) - 1)]            # the fc1-shaped layer
        s = Ld["shape"]
        L = Ld["host"]
        Ms = s.M
        Wh, qw, sw = O.prepare_weights(L.W, L.Q32, s.r, s.g)          # offline, not timed
        xs = I.bf16_bits_to_f32(L.x_bits[:Ms])
        Qb = I.bf16_bits_to_f32(L.Q_bits)
        tc = time.perf_counter()
        (O.linear_a8 if args.a8 else O.linear_asym if args.asym else O.linear)(xs, Qb, Wh, qw, sw, s.r, s.g)
        dt = time.perf_counter() - tc
        try:
            cores = len(os.sched_getaffinity(0))
        except AttributeError:
            cores = os.cpu_count()
        cores = min(cores, int(os.environ.get("OMP_NUM_THREADS", cores)))
        cpu = {"value": 2.0 * Ms * s.N * s.K / dt / 1e12, "unit": "TOPS", "cores": cores, "kind": "oracle",
               "seconds": round(dt, 2),
               "implementation": "NumPy oracle: float64 BLAS matmuls for the rotation and the per-group integer dots, "
                                 "vectorised quantizer; not a hand-written loop nest",
               "sample": f"online part of the NumPy oracle (rotate, quantize, combine; float64 BLAS for the sums) on "
                         f"{Ms} tokens of {s.name} (K={s.K}, N={s.N}), one of the four layers of a step; "
                         f"effective ops 2*{Ms}*N*K; the offline weight preparation is not timed"}
        log(f"oracle on {Ms} tokens of {s.name}: {dt:.1f} s on {cores} cores")

    out = {
        "metric": "effective TOPS of fused rotate+quant+W4A4 linear, FLUX shapes",
        "value": round(value, 3), "unit": "TOPS", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": round(ms_per_step, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": ("fp8 e4m3 or fp6 e2m3 (128 x 128 tiles)" if args.asym else "fp6 e2m3 (large layers) or fp8 e4m3") +
                 " (exact integer codes, fp32 accumulate) + bf16 (fp32 accumulate)", "data": "synthetic",
        "config": {"workload": {"flux": "FLUX.1-dev-shaped block linears, M=4608 tokens, hidden 3072, "
                                        "r=128, g=64: fused QKV (N=9216), out-proj (N=3072), fc1 (N=12288), "
                                        "fc2 (K=12288, N=3072); one dirotq_linear per layer per step",
                                "pixart": "PixArt-Sigma-shaped block linears, M=4096",
                                "small": "M=256, K=N=1152",
                                "sweep": "token sweep on the PixArt fc1 shape, M in {1024..32768}",
                                "ablation": "rank/group grid on the FLUX fc2 shape"}[args.workload],
                   "seed": 0, "effective_ops_per_step": total_ops, "residual_rotation": args.residual_rotation,
                   "activation_quantizer": "int8 per token" if args.a8 else "asymmetric" if args.asym else "symmetric",
                   "shared_input": bool(args.shared_input)},
        "speedup_vs_bf16_gemm": round(bf16_ms / ms_per_step, 4),
        "bf16_gemm_ms_per_step": round(bf16_ms, 4),
        "graph_ms_per_step": None if graph_ms is None else round(graph_ms, 4),
        "roofline": {k: (round(v, 5) if isinstance(v, float) else v) for k, v in roofline.items()},
        "kernels": other,
        "peaks": {"datasheet": {"bf16_tflops": PEAK_BF16_TFLOPS, "fp8_tops": PEAK_FP8_TOPS, "fp6_tops": PEAK_FP6_TOPS,
                                 "hbm_gbs": PEAK_HBM_GBS},
                  "measured_mfma_only": measured_peaks},
        "layers": per_layer,
        "cpu_baseline": cpu,
        "paper_context": "paper reports 2.3x end-to-end speedup and 2.1x memory reduction for FLUX.1-dev on an "
                         "RTX 4090 (whole model, other hardware): context only",
    }
    print(json.dumps(out), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())

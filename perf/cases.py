"""The calls whose speed this repository answers for: the rotated 4-bit linear layer and its variants, over the token
counts, layer shapes, ranks, group sizes and activation formats that its workloads have.

`listed` are fixed representatives, `draw` gives more of the same ranges, `prepare` makes a call's inputs, `run` is
the call, `work` what it cannot do without, `tolerance` how far another correct implementation may be off, and
`exact` the same outputs in 64-bit arithmetic.
"""
import math

import torch

from paper_2605_16732_amd import binding as dq

DEV = "cuda"
# cost of the largest listed case (multiply-adds of rotation and product); no drawn case has more
MAX_MACS = 4608 * 12288 * (12288 + 3072)


def listed():
    return [
        # one DiT linear at a low resolution (16 x 16 latent patches): launch latency counts
        dict(name="linear_small", op="linear", M=256, K=1152, N=1152, r=64, g=64, bias=True),
        # a short text prompt through a hidden-3072 layer: fewer tokens than a tile, odd count
        dict(name="linear_few", op="linear", M=77, K=3072, N=3072, r=128, g=64, bias=True),
        # the MLP's first projection of a 1152-wide block at 1024 px (4096 patches), batch 1
        dict(name="linear_block", op="linear", M=4096, K=1152, N=4608, r=64, g=64, bias=True),
        # the same layer at batch 8
        dict(name="linear_batch", op="linear", M=32768, K=1152, N=4608, r=64, g=64, bias=True),
        # the MLP's first projection of a 3072-wide block, 4096 image + 512 text tokens
        dict(name="linear_fc1", op="linear", M=4608, K=3072, N=12288, r=128, g=64, bias=True),
        # and its second one: the K x K rotation dominates; the largest call
        dict(name="linear_fc2", op="linear", M=4608, K=12288, N=3072, r=128, g=64, bias=True),
        # asymmetric activations (the form the paper's experiments use), a ragged medium token count
        dict(name="asym_out", op="asym", M=1000, K=3072, N=3072, r=128, g=64, bias=True),
        # 8-bit per-token activations, fused QKV of a 1152-wide block
        dict(name="a8_qkv", op="a8", M=4096, K=1152, N=3456, r=64, g=64, bias=True),
        # a down-projection whose activations stay in 16 bits
        dict(name="w4a16_fc2", op="w4a16", M=4096, K=4608, N=1152, r=0, g=64, bias=True),
        # the adaptive-normalisation projection of one conditioning vector
        dict(name="w4a16_vector", op="w4a16", M=1, K=3072, N=9216, r=0, g=64, bias=True),
        # the two halves called on their own (activations quantized by one program part, multiplied by another):
        # smallest groups, fp32 output, nothing a multiple of a tile
        dict(name="split_ragged", op="split", M=1999, K=2080, N=2500, r=32, g=32, bias=False),
        # loading a layer: rotation operand and weight fusion / quantization, with the read-back of the result
        dict(name="load_layer", op="load", M=1, K=1536, N=1536, r=64, g=64, bias=False),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choices(["linear", "asym", "a8", "w4a16", "split", "load"], [8, 3, 3, 3, 2, 1])[0]
    g = rng.choices([64, 32, 128], [6, 1, 2])[0]
    while True:
        K = _log_uniform(rng, 640, 1536 if op == "load" else 12288)   # (loading: 64-bit arithmetic, the listed layer's size)
        K = max(640, K // 128 * 128 if rng.random() < 0.7 else K // 32 * 32)
        r = 0 if op == "w4a16" else rng.choice([0, 32, 64, 64, 128, 128, 256])
        if (K - r) % g == 0:
            break
    N = _log_uniform(rng, 320, 12288)
    N = N // 64 * 64 if rng.random() < 0.75 else N
    if op == "load":
        return dict(op=op, M=1, K=K, N=min(N, 1536), r=r, g=g, bias=False)
    M = _log_uniform(rng, 1, 32768)
    M = min(M, MAX_MACS // (K * (N + (0 if op == "w4a16" else K))))
    if M > 8 and rng.random() < 0.5:
        M = M // 8 * 8
    return dict(op=op, M=M, K=K, N=N, r=r, g=g, bias=rng.random() < 0.5)


# ---- inputs -------------------------------------------------------------------------------------------


def _orthogonal(n, gen):
    return torch.linalg.qr(torch.randn(n, n, generator=gen, dtype=torch.float64))[0]


def _layer(case, seed):
    """Activations with a few outlier channels, a PCA-like orthogonal basis (top-scale channels first, a full mixing of
    each part, a little of everything everywhere), dense weights and a bias; fp32 on the GPU, x in bf16."""
    M, K, N, r = case["M"], case["K"], case["N"], case["r"]
    cpu = torch.Generator().manual_seed(seed)
    gpu = torch.Generator(device=DEV).manual_seed(seed)
    scale = torch.exp(0.5 * torch.randn(K, generator=cpu, dtype=torch.float64))
    scale[torch.randperm(K, generator=cpu)[: 16 if K >= 3072 else 8]] *= 80.0
    scale32 = scale.float().to(DEV)
    x = (torch.randn(M, K, device=DEV, generator=gpu) * scale32).to(torch.bfloat16)
    W = torch.randn(N, K, device=DEV, generator=gpu) / math.sqrt(K)
    bias = torch.randn(N, device=DEV, generator=gpu).to(torch.bfloat16) if case["bias"] else None
    if case["op"] == "w4a16":
        return x, None, W, bias
    order = torch.argsort(scale, descending=True).to(DEV)
    Q = torch.zeros(K, K, device=DEV)
    if r:
        Q[:r, :r] = _orthogonal(r, cpu).float().to(DEV)
    if r < K:
        a, b = _orthogonal((K - r) // 32, cpu).float().to(DEV), _orthogonal(32, cpu).float().to(DEV)
        Q[r:, r:] = torch.kron(a, b)
    v = torch.randn(K, device=DEV, generator=gpu)
    v /= v.norm()
    Q -= torch.outer(2 * v, v @ Q)
    Qc = torch.empty_like(Q)
    Qc[order] = Q
    return x, Qc, W, bias


def prepare(case, seed):
    M, K, N, r, g, op = (case[k] for k in ("M", "K", "N", "r", "g", "op"))
    x, Q, W, bias = _layer(case, seed)
    s = dict(case, x=x, bias=bias)
    if op == "load":
        s.update(W=W, Q=Q)
        return s
    if op == "w4a16":
        # codes and scales of the weights themselves (this format has no rotation)
        codes, sw = _quantize_weights(W, g)
        s["blob"] = dq.import_weights(None, codes, sw, N, K, 0, g)
        s["y"] = torch.empty(M, N, dtype=torch.bfloat16, device=DEV)
        return s
    s["Qt"] = dq.prepare_rotation(Q)
    s["blob"] = dq.prepare_weights(W, Q, r, g)
    if op == "split":
        return s
    size = dq.a8_workspace_bytes(M, K, r) if op == "a8" else dq.workspace_bytes(M, K, r, g)
    s["ws"] = torch.empty(size, dtype=torch.uint8, device=DEV)
    s["y"] = torch.empty(M, N, dtype=torch.bfloat16, device=DEV)
    return s


def run(s):
    op, N, K, r, g = s["op"], s["N"], s["K"], s["r"], s["g"]
    if op == "linear":
        return dq.linear(s["x"], s["Qt"], s["blob"], N, r, g, bias=s["bias"], workspace=s["ws"], out=s["y"])
    if op == "asym":
        return dq.linear_asym(s["x"], s["Qt"], s["blob"], N, r, g, bias=s["bias"], workspace=s["ws"], out=s["y"])
    if op == "a8":
        return dq.linear_a8(s["x"], s["Qt"], s["blob"], N, r, g, bias=s["bias"], workspace=s["ws"], out=s["y"])
    if op == "w4a16":
        return dq.w4a16_gemm(s["x"], s["blob"], N, g, bias=s["bias"], out=s["y"])
    if op == "split":
        xh, xl, sx = dq.rotate_quantize(s["x"], s["Qt"], r, g)
        y = dq.w4a4_gemm(xh, xl, sx, s["blob"], s["M"], N, K, r, g, bias=s["bias"], out_dtype=torch.float32)
        return xh, xl, sx, y
    Qt = dq.prepare_rotation(s["Q"])
    blob = dq.prepare_weights(s["W"], s["Q"], r, g)
    Wh, codes, sw = dq.export_weights(blob, N, K, r, g)
    return Qt, Wh, codes, sw


# ---- what a call cannot do without -----------------------------------------------------------------------


def work(case):
    M, K, N, r, g, op = (case[k] for k in ("M", "K", "N", "r", "g", "op"))
    G = (K - r) // g
    blob = 2 * N * r + N * (K - r) // 2 + 2 * N * G
    if op == "load":
        return dict(bytes=4 * N * K + 4 * K * K + 2 * K * K + 2 * N * r + N * (K - r) + 2 * N * G, flops=2 * N * K * K)
    if op == "w4a16":
        return dict(bytes=2 * M * K + blob + 2 * M * N + 2 * N * case["bias"], flops=2 * M * N * K)
    moved = 2 * M * K + 2 * K * K + blob + 2 * M * N + 2 * N * case["bias"]
    if op == "split":
        moved += 2 * M * N + 2 * (2 * M * r + M * (K - r) // 2 + 2 * M * G)     # fp32 output; written and read again
    return dict(bytes=moved, flops=2 * M * K * K + 2 * M * N * K)


def tolerance(case):
    """About four times what `run` differs by from `exact` rounded to the output's type (listed cases and ten draws)."""
    if case["op"] == "w4a16":
        # products exact, fp32 sums in another order: a bf16 rounding here and there (2.4e-5 and 7.7e-3 seen)
        return dict(rel=1.2e-4, max=3e-2)
    if case["op"] == "load":
        # 64-bit sums in another order: a value next to a rounding boundary (none seen)
        return dict(rel=1e-6, max=1e-2, differ=1e-6)
    # a rotated value next to a rounding boundary (about sqrt(K) 2^-24 of the accumulated magnitude from it) takes the
    # neighbouring code, a scale the neighbouring fp16 number; then the output's own rounding (4e-4, 1.8e-2 and, for
    # the codes themselves, 3e-6 seen)
    return dict(rel=1.6e-3, max=7e-2, differ=2e-5)


# ---- the same in 64 bits ------------------------------------------------------------------------------------


def _scale16(num, div):
    return torch.clamp((num / torch.tensor(div, dtype=torch.float32, device=num.device)), max=65504.0).half()


def _inv(s16):
    s = s16.float()
    return torch.where(s == 0, torch.zeros_like(s), 1.0 / s)


def _quantize_weights(Wl, g):
    """fp32 [N, KL] -> int8 codes [N, KL], fp16 scales [N, G]: scale max|v| / 7, round to nearest even, +-7."""
    v = Wl.view(Wl.shape[0], -1, g)
    sw = _scale16(v.abs().amax(-1), 7.0)
    codes = torch.clamp(torch.round(v * _inv(sw)[..., None]), -7, 7).to(torch.int8)
    return codes.view(Wl.shape[0], -1), sw


def _weights64(Wl, g):
    codes, sw = _quantize_weights(Wl, g)
    return (codes.view(Wl.shape[0], -1, g).double() * sw.double()[..., None]).reshape(Wl.shape[0], -1)


def exact(case, seed):
    M, K, N, r, g, op = (case[k] for k in ("M", "K", "N", "r", "g", "op"))
    x, Q, W, bias = _layer(case, seed)
    b = bias.double() if bias is not None else 0.0
    if op == "w4a16":
        return x.double() @ _weights64(W, g).t() + b
    Wr = (W.double() @ Q.double()).float()
    if op == "load":
        Wh = Wr[:, :r].to(torch.bfloat16)
        codes, sw = _quantize_weights(Wr[:, r:].contiguous(), g)
        return Q.t().to(torch.bfloat16).double(), Wh.double(), codes.to(torch.int64), sw.double()
    v = x.double() @ Q.to(torch.bfloat16).double()
    xh = v[:, :r].float().to(torch.bfloat16)
    y = xh.double() @ Wr[:, :r].to(torch.bfloat16).double().t() + b
    if r == K:
        return y
    vl = v[:, r:].float().contiguous()
    Wl = _weights64(Wr[:, r:].contiguous(), g)
    if op == "a8":
        s = _scale16(vl.abs().amax(-1, keepdim=True), 127.0)
        q = torch.clamp(torch.round(vl * _inv(s)), -127, 127)
        return y + (q.double() * s.double()) @ Wl.t()
    vg = vl.view(M, -1, g)
    if op == "asym":
        lo, hi = vg.amin(-1), vg.amax(-1)
        z = torch.clamp(lo, -65504.0, 65504.0).half()
        s = _scale16(hi - lo, 15.0)
        q = torch.clamp(torch.round((vg - z.float()[..., None]) * _inv(s)[..., None]), 0, 15)
        xq = q.double() * s.double()[..., None] + z.double()[..., None]
        return y + xq.reshape(M, -1) @ Wl.t()
    s = _scale16(vg.abs().amax(-1), 7.0)
    q = torch.clamp(torch.round(vg * _inv(s)[..., None]), -7, 7)
    y = y + (q.double() * s.double()[..., None]).reshape(M, -1) @ Wl.t()
    if op == "split":
        n = q.reshape(M, -1).to(torch.int64)
        n = torch.where(n < 0, 8 - n, n)                     # sign-magnitude nibbles, even channel in the low half
        return xh.double(), (n[:, 0::2] | n[:, 1::2] << 4).to(torch.uint8), s.t().contiguous().double(), y
    return y

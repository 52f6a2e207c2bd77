"""The pipelined W4A8 GEMM (256 x 256 tiles, FP6 planes), forced on every input, against the CPU oracle on identical inputs: one
output, cut tiles, rows that are and are not stored through LDS, odd numbers of 64-channel stages, no 16-bit part, several
tiles per workgroup, both group sizes, the extreme codes in both planes."""
import numpy as np
import pytest
import torch

from oracle import dirotq_oracle as O
from paper_2605_16732_amd import binding as B

from gpu_util import dev, dev_bf16, host_bf16_bits, import_blob

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,r,g,extreme", [
    (1, 1, 64, 0, 64, False), (257, 255, 96, 32, 64, True), (256, 256, 128, 0, 128, True), (300, 520, 1152, 64, 64, False),
    (511, 264, 1120, 32, 64, False), (33, 1032, 2304, 256, 128, False), (4200, 4400, 192, 64, 64, False), (4400, 4104, 64, 0, 64, False),
    (270, 300, 12288, 128, 128, False),
])
def test_matches_oracle(M, N, K, r, g, extreme, monkeypatch):
    """fp32 sums of G products and r / 16 partial sums against a float64 sum: 1e-5 of the largest output; the bf16 output is
    the rounded fp32 one."""
    print(f"[case] w4a8 pipe M={M} N={N} K={K} r={r} g={g}", flush=True)
    monkeypatch.setenv("DIROTQ_W4A8_KERNEL", "pipe")
    rng = np.random.default_rng([M, N, K])
    G = (K - r) // g
    xh = O.round_to_bf16(rng.standard_normal((M, r)).astype(np.float32) * 20)
    Wh = O.round_to_bf16(rng.standard_normal((N, r)).astype(np.float32) * 0.05)
    qx = rng.integers(-127, 128, size=(M, K - r)).astype(np.int32)
    qw = rng.integers(-7, 8, size=(N, K - r)).astype(np.int8)
    if extreme:
        qx, qw = np.where(qx < 0, -127, 127).astype(np.int32), np.where(qw < 0, -7, 7).astype(np.int8)
    sx = rng.lognormal(-3, 1, size=M).astype(np.float16)
    sw = rng.lognormal(-5, 1, size=(N, G)).astype(np.float16)
    bias = O.round_to_bf16(rng.standard_normal(N).astype(np.float32))
    want, _ = O.combine_a8(xh, qx, sx, Wh, qw, sw, g, bias)
    sm = np.where(qx < 0, 0x80 - qx, qx).astype(np.uint8).reshape(M, (K - r) // 32, 16, 2)
    x8 = np.ascontiguousarray(sm.transpose(0, 1, 3, 2)).reshape(M, K - r)      # blocks of 32: even channels, odd ones
    args = (dev_bf16(O.bf16_bits(xh)) if r else None, dev(x8), dev(sx), import_blob(Wh, qw, sw, N, K, r, g), M, N, K, r, g)
    bias_d = dev_bf16(O.bf16_bits(bias))
    yf = B.w4a8_gemm(*args, bias=bias_d, out_dtype=torch.float32).cpu().numpy()
    yb = B.w4a8_gemm(*args, bias=bias_d, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    assert np.abs(yf - want).max() <= 1e-5 * np.abs(want).max()
    np.testing.assert_array_equal(host_bf16_bits(yb).astype(np.int32), O.bf16_bits(O.round_to_bf16(yf)).astype(np.int32))

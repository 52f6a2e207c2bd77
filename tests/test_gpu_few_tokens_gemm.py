"""The few-token schedules of the W4A4 GEMM (K split over the waves of a workgroup; 64 x 64 and 32 x 32 outputs), with
symmetric and asymmetric activation codes, each forced on every input, against the CPU oracle on identical inputs: one
output, one item of the K axis, fewer items than waves, several items for every wave, an odd number of 64-channel pieces,
groups of two pieces, cut tiles."""
import numpy as np
import pytest
import torch

from oracle import dirotq_oracle as O
from paper_2605_16732_amd import binding as B

from gpu_util import pack_codes, dev, dev_bf16, import_blob

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", ["skinny32", "skinny64"])
@pytest.mark.parametrize("M,N,K,r,g", [
    (1, 1, 64, 0, 64), (1, 33, 32, 0, 32), (31, 70, 96, 32, 32), (33, 32, 192, 64, 128), (65, 129, 1152, 64, 64),
    (130, 1024, 288, 32, 128), (1000, 1160, 160, 32, 64), (700, 2500, 96, 32, 32),
    (40, 65, 2080, 32, 32), (100, 130, 2112, 64, 64), (70, 100, 3232, 32, 128),              # 4 to 8 items a wave
])
def test_few_token_schedules_match_oracle(M, N, K, r, g, tiles, monkeypatch):
    """fp32 sums of at most G + r/16 partial terms per wave and 8 waves against a float64 sum: 1e-5 of the largest output
    (2e-5 with zero-points: six products of exact bf16 pieces per group more)."""
    print(f"[case] few-token w4a4 M={M} N={N} K={K} r={r} g={g} {tiles}", flush=True)
    monkeypatch.setenv("DIROTQ_W4A4_KERNEL", tiles)
    rng = np.random.default_rng([M, N, K])
    G = (K - r) // g
    xh = O.round_to_bf16(rng.standard_normal((M, r)).astype(np.float32) * 20)
    Wh = O.round_to_bf16(rng.standard_normal((N, r)).astype(np.float32) * 0.05)
    qx = rng.integers(-7, 8, size=(M, K - r)).astype(np.int8)
    ux = rng.integers(0, 16, size=(M, K - r)).astype(np.int8)
    qw = rng.integers(-7, 8, size=(N, K - r)).astype(np.int8)
    sx = rng.lognormal(-1, 1, size=(M, G)).astype(np.float16)
    zx = rng.standard_normal((M, G)).astype(np.float16)
    sw = rng.lognormal(-5, 1, size=(N, G)).astype(np.float16)
    bias = O.round_to_bf16(rng.standard_normal(N).astype(np.float32))
    blob = import_blob(Wh, qw, sw, N, K, r, g)
    xh_d, bias_d = dev_bf16(O.bf16_bits(xh)) if r else None, dev_bf16(O.bf16_bits(bias))
    sx_d, zx_d = dev(np.ascontiguousarray(sx.T)), dev(np.ascontiguousarray(zx.T))
    want, _ = O.combine(xh, qx, sx, Wh, qw, sw, g, bias)
    got = B.w4a4_gemm(xh_d, dev(pack_codes(qx)), sx_d, blob, M, N, K, r, g, bias=bias_d, out_dtype=torch.float32)
    assert np.abs(got.cpu().numpy() - want).max() <= 1e-5 * np.abs(want).max()
    want, _ = O.combine_asym(xh, ux, sx, zx, Wh, qw, sw, g, bias)
    packed = (ux[:, 0::2] | (ux[:, 1::2] << 4)).astype(np.uint8)
    got = B.w4a4_gemm_asym(xh_d, dev(packed), sx_d, zx_d, blob, M, N, K, r, g, bias=bias_d, out_dtype=torch.float32)
    assert np.abs(got.cpu().numpy() - want).max() <= 2e-5 * np.abs(want).max()


@pytest.mark.parametrize("tiles", ["skinny32", "skinny64"])
def test_zero_point_term_is_multiplied_out(tiles, monkeypatch):
    """All codes 0, one group: the output is z s_w sum(q_w), as six products of bf16 pieces in one fp32 accumulator.  The
    numbers make the last one (z2 c3) as large as it gets, 2^-22.3 of the term.  With it the error is that of the sum and of
    its result, at most 2^-24 each; without it 2.26 x 2^-24 were seen."""
    print(f"[case] few-token w4a4 zero-point term {tiles}", flush=True)
    monkeypatch.setenv("DIROTQ_W4A4_KERNEL", tiles)
    qw = np.zeros((1, 64), np.int8)
    qw[0, :58], qw[0, 58] = 7, 3
    z, sw = np.float16(1.0068359375), np.float16(1.2568359375)
    blob = import_blob(np.zeros((1, 0), np.float32), qw, np.full((1, 1), sw), 1, 64, 0, 64)
    y = B.w4a4_gemm_asym(None, torch.zeros((1, 32), dtype=torch.uint8, device="cuda"), dev(np.ones((1, 1), np.float16)),
                         dev(np.full((1, 1), z)), blob, 1, 1, 64, 0, 64, out_dtype=torch.float32)
    want = float(z) * float(sw) * 409.0
    assert abs(float(y) - want) <= 2.0 ** -23 * want

"""The pipelined schedule of the W4A4 GEMM (256 x 256 and 256 x 128 tiles, one kernel) against the CPU oracle on
identical inputs: tiles that are cut in either direction, one stage of K only, an odd number of 64-channel stages, no
16-bit branch and a long one, all group sizes, and a launch whose workgroups take tiles of both sizes one after the
other."""
import numpy as np
import pytest
import torch

from oracle import dirotq_oracle as O
from paper_2605_16732_amd import binding as B

from gpu_util import pack_codes, dev, dev_bf16, host_bf16_bits, import_blob

pytestmark = pytest.mark.gpu


def _compare(M, N, K, r, g, use_bias):
    """fp32 sums of at most G + r/16 + 1 partial terms, each exact up to its own rounding, against a float64 sum: 1e-5
    of the largest output per element, as for the other schedules; the bf16 output is the rounded fp32 one."""
    print(f"[case] pipelined w4a4 M={M} N={N} K={K} r={r} g={g} bias={use_bias}", flush=True)
    rng = np.random.default_rng([M, N, K, r, g])
    G = (K - r) // g
    xh = O.round_to_bf16(rng.standard_normal((M, r)).astype(np.float32) * 20)
    Wh = O.round_to_bf16(rng.standard_normal((N, r)).astype(np.float32) * 0.05)
    qx = rng.integers(-7, 8, size=(M, K - r)).astype(np.int8)
    qw = rng.integers(-7, 8, size=(N, K - r)).astype(np.int8)
    sx = rng.lognormal(-1, 1, size=(M, G)).astype(np.float16)
    sw = rng.lognormal(-5, 1, size=(N, G)).astype(np.float16)
    bias = O.round_to_bf16(rng.standard_normal(N).astype(np.float32)) if use_bias else None
    y32, _ = O.combine(xh, qx, sx, Wh, qw, sw, g, bias)
    blob = import_blob(Wh, qw, sw, N, K, r, g)
    args = (dev_bf16(O.bf16_bits(xh)) if r else None, dev(pack_codes(qx)), dev(np.ascontiguousarray(sx.T)), blob, M, N, K,
            r, g)
    bias_d = dev_bf16(O.bf16_bits(bias)) if use_bias else None
    yf = B.w4a4_gemm(*args, bias=bias_d, out_dtype=torch.float32).cpu().numpy()
    yb = B.w4a4_gemm(*args, bias=bias_d, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    assert np.abs(yf - y32).max() <= 1e-5 * np.abs(y32).max()
    np.testing.assert_array_equal(host_bf16_bits(yb).astype(np.int32),
                                  O.bf16_bits(O.round_to_bf16(yf)).astype(np.int32))


@pytest.mark.parametrize("tiles", ["large", "small"])
@pytest.mark.parametrize("M,N,K,r,g,use_bias", [
    (1, 1, 64, 0, 64, False), (256, 256, 64, 0, 64, True), (257, 255, 192, 0, 64, False), (127, 520, 320, 64, 64, True),
    (129, 264, 352, 96, 128, True), (300, 136, 1152, 64, 64, True), (255, 257, 96, 32, 32, False),
    (385, 300, 160, 32, 32, True), (64, 512, 512, 256, 128, False),
])
def test_pipelined_tiles_match_oracle(M, N, K, r, g, use_bias, tiles, monkeypatch):
    monkeypatch.setenv("DIROTQ_W4A4_KERNEL", tiles)
    _compare(M, N, K, r, g, use_bias)


def test_workgroups_take_tiles_of_both_sizes(monkeypatch):
    """19 x 15 tiles of 256 x 256 on 256 CUs: the plan is one round of them and the last tokens in half-size tiles;
    with all tiles small, workgroups take two or three of them in a row (the stage stream crosses tiles)."""
    for tiles in ("pipe", "small"):
        monkeypatch.setenv("DIROTQ_W4A4_KERNEL", tiles)
        _compare(4700, 3592, 224, 32, 64, True)

"""The 128 x 128 tiles of the W4A4 GEMM against the CPU oracle on identical inputs: tiles cut in either direction, one to five stages
of 64 channels over the two parts of K (an odd one alone, a last one of 32 channels), a 16-bit branch of one to 18 passes,
none and nothing else, rows of y of every alignment, both kinds of code, all group sizes."""
import numpy as np
import pytest
import torch

from oracle import dirotq_oracle as O
from paper_2605_16732_amd import binding as B

from gpu_util import dev, dev_bf16, host_bf16_bits, import_blob, pack_codes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("asym", [False, True])
@pytest.mark.parametrize("M,N,K,r,g,use_bias", [
    (1, 1, 64, 0, 64, True), (33, 127, 32, 0, 32, False), (128, 128, 128, 0, 64, True), (129, 130, 192, 0, 64, False),
    (127, 132, 256, 128, 128, True), (40, 129, 352, 32, 64, True), (257, 136, 160, 64, 32, False), (96, 258, 288, 32, 32, True),
    (300, 260, 416, 32, 128, True), (65, 124, 96, 96, 64, True), (130, 257, 1152, 64, 64, True), (31, 384, 672, 32, 128, False),
    # long 16-bit parts: passes of 64 channels, a last one of 32, and nothing else
    (40, 129, 352, 288, 64, True), (129, 130, 416, 320, 32, False), (257, 136, 704, 576, 128, True), (100, 260, 992, 960, 32, True),
    (130, 127, 288, 288, 64, False), (33, 140, 320, 320, 64, True), (200, 129, 672, 672, 32, True), (128, 128, 1152, 1152, 128, True),
    # more than one tile per CU without 4-bit channels
    (2100, 2201, 96, 96, 64, True), (4200, 1100, 192, 192, 32, False),
])
def test_tiles_match_oracle(M, N, K, r, g, use_bias, asym, monkeypatch):
    """fp32 sums of at most G + r/16 + 1 partial terms (asymmetric: and six exact products for each group), each exact up to its
    own rounding, against a float64 sum: 1e-5 of the largest output per element, asymmetric 2e-5 (the zero-point terms
    cancel against the codes'), as for the other schedules; the bf16 output is the rounded fp32 one."""
    monkeypatch.setenv("DIROTQ_W4A4_KERNEL", "tile")
    print(f"[case] w4a4 tile M={M} N={N} K={K} r={r} g={g} bias={use_bias} asym={asym}", flush=True)
    rng = np.random.default_rng([M, N, K, r, g])
    G = (K - r) // g
    xh = O.round_to_bf16(rng.standard_normal((M, r)).astype(np.float32) * 20)
    Wh = O.round_to_bf16(rng.standard_normal((N, r)).astype(np.float32) * 0.05)
    qw = rng.integers(-7, 8, size=(N, K - r)).astype(np.int8)
    sx = rng.lognormal(-1, 1, size=(M, G)).astype(np.float16)
    zx = (rng.standard_normal((M, G)) * 3).astype(np.float16)
    sw = rng.lognormal(-5, 1, size=(N, G)).astype(np.float16)
    bias = O.round_to_bf16(rng.standard_normal(N).astype(np.float32)) if use_bias else None
    qx = rng.integers(0 if asym else -7, 16 if asym else 8, size=(M, K - r)).astype(np.int8)
    dq = lambda q, s: (q.reshape(q.shape[0], G, g).astype(np.float64) * s.astype(np.float64)[..., None])
    xl = dq(qx, sx) + (zx.astype(np.float64)[..., None] if asym else 0.0)
    want = xh.astype(np.float64) @ Wh.astype(np.float64).T + xl.reshape(M, K - r) @ dq(qw, sw).reshape(N, K - r).T
    if bias is not None:
        want = want + bias.astype(np.float64)
    blob = import_blob(Wh, qw, sw, N, K, r, g)
    codes = (qx[:, 0::2] | (qx[:, 1::2] << 4)).astype(np.uint8) if asym else pack_codes(qx) if r < K else np.zeros((M, 0), np.uint8)
    four_bit = (dev(codes), dev(np.ascontiguousarray(sx.T))) + ((dev(np.ascontiguousarray(zx.T)),) if asym else ())
    args = (dev_bf16(O.bf16_bits(xh)) if r else None,) + four_bit + (blob, M, N, K, r, g)
    bias_d = dev_bf16(O.bf16_bits(bias)) if use_bias else None
    f = B.w4a4_gemm_asym if asym else B.w4a4_gemm
    yf = f(*args, bias=bias_d, out_dtype=torch.float32).cpu().numpy()
    yb = f(*args, bias=bias_d, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    assert np.abs(yf - want).max() <= (2e-5 if asym else 1e-5) * np.abs(want).max()
    np.testing.assert_array_equal(host_bf16_bits(yb).astype(np.int32), O.bf16_bits(O.round_to_bf16(yf)).astype(np.int32))

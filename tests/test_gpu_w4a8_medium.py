"""The medium schedule of the W4A8 GEMM (1, 2 and 4 token tiles per workgroup, each forced) against a float64 product of
the same numbers: cut tiles, an odd number of output channels, one stage, odd numbers of stages, a last stage of half the
channels, no 8-bit part, 16-bit parts of half a 64-channel piece, several and none."""
import numpy as np
import pytest
import torch

from paper_2605_16732_amd import binding as B

from gpu_util import dev, dev_bf16, import_blob
from oracle import dirotq_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [1, 2, 4])
@pytest.mark.parametrize("M,N,K,r,g", [
    (300, 2049, 416, 32, 32), (300, 2050, 448, 0, 64), (300, 2049, 416, 32, 128), (300, 2050, 512, 512, 64),
    (1030, 1153, 608, 160, 32), (1030, 1160, 640, 64, 64),
    (2050, 1153, 1120, 96, 128), (2050, 1153, 1184, 32, 32), (2050, 1160, 1152, 256, 64),
])
def test_medium_matches_float64(M, N, K, r, g, tiles, monkeypatch):
    """Group sums are exact (whole numbers below 2^24); an output is G scaled ones, r products, a token scale and a bias in
    fp32: at most G + r + 4 roundings of 2^-24 of the sum of the magnitudes.  The bf16 output is the rounded fp32 one."""
    print(f"[case] w4a8 medium M={M} N={N} K={K} r={r} g={g} tiles={tiles}", flush=True)
    monkeypatch.setenv("DIROTQ_W4A8_KERNEL", f"medium{tiles}")
    rng = np.random.default_rng([M, N, K, r])
    G = (K - r) // g
    xh = O.round_to_bf16(rng.standard_normal((M, r)).astype(np.float32) * 20)
    Wh = O.round_to_bf16(rng.standard_normal((N, r)).astype(np.float32) * 0.05)
    qx = rng.integers(-127, 128, size=(M, K - r)).astype(np.int32)
    qw = rng.integers(-7, 8, size=(N, K - r)).astype(np.int8)
    sx = rng.lognormal(-3, 1, size=M).astype(np.float16)
    sw = rng.lognormal(-5, 1, size=(N, G)).astype(np.float16)
    bias = O.round_to_bf16(rng.standard_normal(N).astype(np.float32))
    sm = np.where(qx < 0, 0x80 - qx, qx).astype(np.uint8).reshape(M, (K - r) // 32, 16, 2)
    x8 = np.ascontiguousarray(sm.transpose(0, 1, 3, 2)).reshape(M, K - r)      # blocks of 32: even channels, odd ones
    xd = torch.from_numpy(qx.astype(np.float64) * sx.astype(np.float64)[:, None])
    wd = torch.from_numpy(qw.astype(np.float64) * np.repeat(sw.astype(np.float64), g, axis=1).reshape(N, K - r))
    xh64, wh64, b64 = (torch.from_numpy(a).double() for a in (xh, Wh, bias))
    want = xh64 @ wh64.T + xd @ wd.T + b64
    # a group's sum is exact, so only its magnitude counts, not that of its products
    mag = xh64.abs() @ wh64.abs().T + b64.abs()
    for j in range(G):
        mag += (xd[:, j * g:(j + 1) * g] @ wd[:, j * g:(j + 1) * g].T).abs()
    low = r < K
    args = (dev_bf16(O.bf16_bits(xh)) if r else None, dev(x8) if low else None, dev(sx) if low else None,
            import_blob(Wh, qw, sw, N, K, r, g), M, N, K, r, g)
    bias_d = dev_bf16(O.bf16_bits(bias))
    yf = B.w4a8_gemm(*args, bias=bias_d, out_dtype=torch.float32)
    yb = B.w4a8_gemm(*args, bias=bias_d, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    yf, yb = yf.cpu(), yb.cpu()
    assert bool(((yf.double() - want).abs() <= (G + r + 4) * 2.0 ** -24 * mag).all())
    assert torch.equal(yb, yf.bfloat16())

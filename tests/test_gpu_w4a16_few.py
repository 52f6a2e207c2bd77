"""The W4A16 streams over the packed weights (up to 8 tokens, 9 to 32 in workgroups of 32 or 48 channels, two launches beyond)
against a float64 product of the same numbers: the token counts at each switch, cut channel tiles, an odd number of
channels, one panel, a last panel of one group, more panels than the ring holds, all group sizes."""
import numpy as np
import pytest
import torch

from paper_2605_16732_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,g", [(M, N, K, g) for M in (1, 8, 9, 16, 17, 32) for N, K, g in
                                     ((33, 32, 32), (70, 544, 32), (257, 2624, 64), (129, 1152, 128), (8201, 608, 32), (9216, 576, 64),
                                      (8250, 2688, 128))] + [(40, 100, 4672, 64), (64, 33, 4640, 32)])
def test_matches_float64(M, N, K, g):
    """Each output is a sum of K fp32 products and G scaled ones: K + G roundings of at most 2^-24 of the sum of the
    magnitudes; the bf16 output is the rounded fp32 one."""
    print(f"[case] w4a16 few M={M} N={N} K={K} g={g}", flush=True)
    rng = np.random.default_rng([M, N, K, g])
    G = K // g
    x = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).bfloat16()
    qw = rng.integers(-7, 8, size=(N, K)).astype(np.int8)
    sw = rng.lognormal(-4, 0.7, size=(N, G)).astype(np.float16)
    bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32)).bfloat16()
    blob = B.import_weights(None, torch.from_numpy(qw).cuda(), torch.from_numpy(sw).cuda(), N, K, 0, g)
    w = torch.from_numpy(qw.astype(np.float64) * np.repeat(sw.astype(np.float64), g, axis=1))
    want = x.double() @ w.T + bias.double()
    bound = (K + G + 8) * 2.0 ** -24 * (x.double().abs() @ w.T.abs() + bias.double().abs())
    args = (x.cuda(), blob, N, g)
    yf = B.w4a16_gemm(*args, bias=bias.cuda(), out_dtype=torch.float32)
    yb = B.w4a16_gemm(*args, bias=bias.cuda(), out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    assert bool(((yf.cpu().double() - want).abs() <= bound).all())
    assert torch.equal(yb, yf.bfloat16())

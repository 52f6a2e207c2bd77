"""Extreme magnitudes through the three activation quantizers (Q = I, so the rotation is exact and
the GPU must reproduce the oracle bit for bit): scales that saturate at the largest fp16 number,
scales that are fp16 subnormals or round to zero, and a token that mixes both ranges.  The rows are repeated up to the
token counts at which the launcher takes each of its kernels (on 256 CUs: few tokens, 128 x 64 with K in two halves,
128 x 128, 256 x 128, 256 x 256, and with K = 32 mod 64 the 128 x 128 and 256 x 128 tiles of 32-channel stages)."""
import sys

import numpy as np
import pytest
import torch

from oracle import dirotq_oracle as O
from paper_2605_16732_amd import binding as B

from gpu_util import dev, dev_bf16, gpu_rotate_quantize, host_f16
from test_gpu_parity_a8 import gpu_rq_a8
from test_gpu_parity_asym import gpu_rq_asym

pytestmark = pytest.mark.gpu


def _rows(K):
    rng = np.random.default_rng(71)
    x = np.zeros((6, K), np.float32)
    x[0] = rng.standard_normal(K) * 1e37                       # amax / 7 far above 65504: scale saturates
    x[1] = rng.standard_normal(K) * 2.0 ** -22                 # fp16-subnormal scales
    x[2] = rng.standard_normal(K) * 2.0 ** -27                 # scales round to zero: all codes 0
    x[3] = rng.standard_normal(K)
    x[3, ::37] = 3e4 * 7                                       # a few channels right at the saturation edge
    x[4, : K // 2] = rng.standard_normal(K // 2) * 1e30        # huge and tiny groups in one token
    x[4, K // 2:] = rng.standard_normal(K // 2) * 2.0 ** -20
    x[5] = np.abs(rng.standard_normal(K)) * 1e36 + 1e36        # one-sided huge values (asymmetric zero-point saturates)
    return O.round_to_bf16(x)


SIZES = [(6, 256), (7000, 256), (9000, 256), (21000, 256), (33000, 256), (6, 288), (5000, 288), (7000, 288)]


def _tokens(M, K):
    """M tokens, the six rows in turn; and how to bring the oracle's result for the six to M tokens."""
    x = _rows(K)
    idx = np.arange(M) % len(x)
    return x, x[idx], idx


@pytest.mark.parametrize("M,K", SIZES)
@pytest.mark.parametrize("g", [32, 64, 128])
def test_extreme_magnitudes_symmetric(g, M, K):
    r = K - 256
    x, xm, idx = _tokens(M, K)
    print(f"[case] extremes symmetric M={M} K={K} r={r} g={g}", flush=True)
    Qt = B.prepare_rotation(dev(np.eye(K, dtype=np.float32)))
    _, qx_r, sx_r = O.split_quantize(x, r, g)
    _, (_, qx_g, sx_g) = gpu_rotate_quantize(O.bf16_bits(xm), Qt, r, g)
    assert float(sx_r[0].astype(np.float32).max()) == 65504.0 and not qx_r[2].any()
    np.testing.assert_array_equal(sx_g.view(np.uint16), sx_r.view(np.uint16)[idx])
    np.testing.assert_array_equal(qx_g, qx_r[idx])


@pytest.mark.parametrize("M,K", SIZES)
@pytest.mark.parametrize("g", [32, 64, 128])
def test_extreme_magnitudes_asymmetric(g, M, K):
    r = K - 256
    x, xm, idx = _tokens(M, K)
    print(f"[case] extremes asymmetric M={M} K={K} r={r} g={g}", flush=True)
    Qt = B.prepare_rotation(dev(np.eye(K, dtype=np.float32)))
    _, qx_r, sx_r, zx_r = O.split_quantize_asym(x, r, g)
    _, (_, qx_g, sx_g, zx_g) = gpu_rq_asym(O.bf16_bits(xm), Qt, r, g)
    assert float(zx_r[5].astype(np.float32).min()) == 65504.0            # zero-point saturates
    np.testing.assert_array_equal(sx_g.view(np.uint16), sx_r.view(np.uint16)[idx])
    np.testing.assert_array_equal(zx_g.view(np.uint16), zx_r.view(np.uint16)[idx])
    np.testing.assert_array_equal(qx_g, qx_r[idx])


@pytest.mark.parametrize("M,K", SIZES)
def test_extreme_magnitudes_int8_tokens(M, K):
    r = K - 256
    x, xm, idx = _tokens(M, K)
    print(f"[case] extremes int8 M={M} K={K} r={r}", flush=True)
    Qt = B.prepare_rotation(dev(np.eye(K, dtype=np.float32)))
    _, qx_r, sx_r = O.split_quantize_a8(x, r)
    _, (_, qx_g, sx_g) = gpu_rq_a8(O.bf16_bits(xm), Qt, r)
    assert float(sx_r[0]) == 65504.0 and not qx_r[2].any()
    np.testing.assert_array_equal(sx_g.view(np.uint16), sx_r.view(np.uint16)[idx])
    np.testing.assert_array_equal(qx_g, qx_r[idx])


@pytest.mark.parametrize("M,K,g", [
    (8, 256, 64), (8, 256, 128), (8, 288, 32), (7000, 256, 64), (9000, 256, 64), (5000, 288, 32), (7000, 288, 32),
    (21000, 256, 64), (33000, 256, 64),
])
def test_a_token_of_nan_gets_scale_zero_in_every_kernel(M, K, g):
    """One NaN makes all rotated channels of its token NaN.  The absolute maximum ignores them, so the symmetric and the
    8-bit scale are 0 and the codes the lower bound, in the few-token kernel as in the tiled ones that the larger token
    counts reach; the other tokens do not change."""
    print(f"[case] NaN token M={M} K={K} g={g}", flush=True)
    x = O.round_to_bf16(np.random.default_rng(M).standard_normal((M, K)).astype(np.float32))
    Qt = B.prepare_rotation(dev(np.eye(K, dtype=np.float32)))
    clean = B.rotate_quantize(dev_bf16(O.bf16_bits(x)), Qt, 0, g) + B.rotate_quantize_a8(dev_bf16(O.bf16_bits(x)), Qt, 0)
    x[M // 2, 5] = np.nan
    bad = B.rotate_quantize(dev_bf16(O.bf16_bits(x)), Qt, 0, g) + B.rotate_quantize_a8(dev_bf16(O.bf16_bits(x)), Qt, 0)
    torch.cuda.synchronize()
    others = np.arange(M) != M // 2
    for i, what in ((1, "codes"), (2, "scales"), (4, "8-bit codes"), (5, "8-bit scales")):
        a, b = (host_f16(v).T if "scales" in what else v.cpu().numpy() for v in (clean[i], bad[i]))
        np.testing.assert_array_equal(b[others], a[others], err_msg=what)
        assert (b[M // 2] == (0 if "scales" in what else 0xFF)).all(), what

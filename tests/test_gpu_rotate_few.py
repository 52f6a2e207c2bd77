"""The few-token rotation + quantization kernel (64 x 32, 64 x 64, 64 x 96 and 128 x 32 tiles, K split over the waves of a
workgroup) and the tiled kernels beyond it against the CPU oracle.  With a signed permutation as basis the rotation is
exact in any order, so bf16 part, codes, scales and zero-points must be equal bit for bit.  The launcher chooses by size;
the comments name its choice on 256 CUs (for the 4-bit quantizers)."""
import numpy as np
import pytest
import torch

from oracle import dirotq_oracle as O
from paper_2605_16732_amd import binding as B

from gpu_util import dev, dev_bf16, gpu_rotate_quantize, host_bf16_bits, host_f16

pytestmark = pytest.mark.gpu

CASES = [
    (1, 32, 0, 32), (33, 32, 32, 64), (5, 96, 32, 64), (32, 160, 64, 32), (97, 288, 96, 64), (31, 2080, 32, 64),
    (640, 1152, 64, 64), (641, 1152, 64, 32), (1300, 768, 32, 32), (300, 1152, 128, 128), (40, 384, 32, 32),
    (1000, 1152, 64, 64), (1343, 1152, 64, 32), (4000, 288, 32, 64),                       # 64 x 96
    (5000, 288, 32, 32), (4033, 288, 32, 64), (3000, 288, 32, 128), (6200, 224, 64, 32),     # tiled, 128 x 128, 32-channel stages
    (7001, 288, 32, 32), (6500, 288, 32, 64), (7001, 288, 32, 128), (7001, 352, 96, 64),     # tiled, 256 x 128, 32-channel stages
    (2300, 768, 64, 64),                                                                   # tiled, K in two halves
]


def _inputs(M, K):
    rng = np.random.default_rng([M, K])
    Q = np.zeros((K, K), np.float32)
    Q[rng.permutation(K), np.arange(K)] = rng.choice([-1.0, 1.0], size=K)
    x = O.round_to_bf16((rng.standard_normal((M, K)) * rng.lognormal(0, 1.5, size=(1, K))).astype(np.float32))
    x[M // 2, :] = 0.0                                   # an all-zero token: scale 0, codes 0
    return x, Q


@pytest.mark.parametrize("M,K,r,g", CASES)
def test_codes_and_scales_are_exact(M, K, r, g):
    print(f"[case] rotate few M={M} K={K} r={r} g={g}", flush=True)
    x, Q = _inputs(M, K)
    Qt = B.prepare_rotation(dev(Q))
    xhat = O.rotate(x, Q)
    _, (xh, qx, sx) = gpu_rotate_quantize(O.bf16_bits(x), Qt, r, g)
    xh_r, qx_r, sx_r = O.split_quantize(xhat, r, g)
    np.testing.assert_array_equal(xh, xh_r)
    if r == K:
        return
    np.testing.assert_array_equal(sx.view(np.uint16), sx_r.view(np.uint16))
    np.testing.assert_array_equal(qx, qx_r)
    xh_a, xl_a, sx_a, zx_a = B.rotate_quantize_asym(dev_bf16(O.bf16_bits(x)), Qt, r, g)
    torch.cuda.synchronize()
    xh_r, qx_r, sx_r, zx_r = O.split_quantize_asym(xhat, r, g)
    p = xl_a.cpu().numpy()
    q = np.stack([p & 15, p >> 4], axis=-1).reshape(M, K - r)
    np.testing.assert_array_equal(q, qx_r)
    np.testing.assert_array_equal(host_f16(sx_a).T.view(np.uint16), sx_r.view(np.uint16))
    np.testing.assert_array_equal(host_f16(zx_a).T.view(np.uint16), zx_r.view(np.uint16))
    np.testing.assert_array_equal(host_bf16_bits(xh_a), O.bf16_bits(xh_r))


@pytest.mark.parametrize("M,K,r", [(1, 32, 0), (33, 160, 64), (130, 1152, 96), (250, 1184, 128), (3000, 288, 32),
                                   (7001, 288, 64)])
def test_8_bit_codes_are_exact(M, K, r):
    print(f"[case] rotate few a8 M={M} K={K} r={r}", flush=True)
    x, Q = _inputs(M, K)
    xh, x8, sx = B.rotate_quantize_a8(dev_bf16(O.bf16_bits(x)), B.prepare_rotation(dev(Q)), r)
    torch.cuda.synchronize()
    xh_r, qx_r, sx_r = O.split_quantize_a8(O.rotate(x, Q), r)
    b = x8.cpu().numpy().astype(np.int32).reshape(M, (K - r) // 32, 2, 16)   # blocks of 32: even channels, odd ones
    q = np.where(b & 0x80, -(b & 0x7F), b).transpose(0, 1, 3, 2).reshape(M, K - r)
    np.testing.assert_array_equal(q, qx_r)
    np.testing.assert_array_equal(host_f16(sx).view(np.uint16), np.asarray(sx_r).reshape(-1).view(np.uint16))
    np.testing.assert_array_equal(host_bf16_bits(xh), O.bf16_bits(xh_r))

"""The per-token 8-bit quantizer, one and four waves per token: with the identity as basis the rotated values are the bf16
inputs themselves, so codes and scales must equal the oracle's bit for bit.  One 32-channel block, rows that end inside
the lanes' stride, the token counts on both sides of the switch, a token of zeros, ties."""
import numpy as np
import pytest
import torch

from oracle import dirotq_oracle as O
from paper_2605_16732_amd import binding as B

from gpu_util import dev_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,r", [(1, 32, 0), (3, 1152, 64), (2047, 96, 0), (2048, 608, 32), (2051, 32, 0), (2050, 2176, 64)])
def test_codes_and_scales_are_the_oracles(M, K, r):
    print(f"[case] a8 quantizer M={M} K={K} r={r}", flush=True)
    rng = np.random.default_rng([M, K])
    x = O.round_to_bf16((rng.standard_normal((M, K)) * rng.lognormal(0, 1, size=(M, 1))).astype(np.float32))
    x[M // 2] = 0.0
    if M > 1:                                              # scale 1: codes are the values, halves round to even
        x[0] = np.clip(rng.integers(-254, 255, size=K) * 0.5, -63.5, 63.5)
        x[0, r] = 127.0
    codes, scales = O.quantize_tokens_int8(x[:, r:])
    _, x8, sx = B.rotate_quantize_a8(dev_bf16(O.bf16_bits(x)), dev_bf16(O.bf16_bits(np.eye(K, dtype=np.float32))), r)
    torch.cuda.synchronize()
    q = codes.astype(np.int32)
    sm = np.where(q < 0, 0x80 - q, q).astype(np.uint8).reshape(M, (K - r) // 32, 16, 2)
    np.testing.assert_array_equal(x8.cpu().numpy(), sm.transpose(0, 1, 3, 2).reshape(M, K - r))
    np.testing.assert_array_equal(sx.cpu().numpy().view(np.uint16), scales.view(np.uint16))

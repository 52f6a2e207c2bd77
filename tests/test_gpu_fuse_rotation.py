"""The fp64 weight fusion W Q: whole numbers whose sums are exact in bf16, read back through the 16-bit part, so that every
output must be equal.  Cut row tiles, fewer 16-channel runs of K than waves, numbers of runs that are no multiple of four."""
import numpy as np
import pytest
import torch

from paper_2605_16732_amd import binding as B

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [(1, 32), (31, 32), (33, 96), (64, 160), (100, 288), (257, 1120), (1000, 1536)])
def test_whole_numbers_are_exact(N, K):
    print(f"[case] fuse N={N} K={K}", flush=True)
    rng = np.random.default_rng([N, K])
    W = rng.integers(-3, 4, size=(N, K)).astype(np.float32)
    Q = np.zeros((K, K), np.float32)
    for _ in range(8):                                     # at most eight terms of 3 x 3: below 2^8
        Q[rng.integers(0, K, size=K), np.arange(K)] = rng.integers(-3, 4, size=K)
    blob = B.prepare_weights(dev(W), dev(Q), K, 32)
    Wh, _, _ = B.export_weights(blob, N, K, K, 32)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(Wh.float().cpu().numpy(), (W.astype(np.float64) @ Q).astype(np.float32))

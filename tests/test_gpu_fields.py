"""Whole W4A4 layers whose kernel A hands the codes over in field form, against the two halves called on their own (nibbles): the
same codes, scales and sums in the same order, so the outputs are equal bit for bit.  Every form of kernel A (few tokens: always nibbles,
K in two halves, 128 x 128, fed by copies, 256 x 256, with a last stage of 32 channels) and every kernel B that reads the field form,
all group sizes, split points inside a tile, asymmetric codes (always nibbles), cut tiles."""
import math

import pytest
import torch

from paper_2605_16732_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule,asym", [("tile", False), ("tile", True), ("large", False), ("small", False)])
@pytest.mark.parametrize("M,K,N,r,g", [
    (1, 640, 96, 0, 64), (37, 640, 320, 64, 64), (70, 704, 136, 128, 64), (33, 1280, 100, 128, 128), (300, 672, 130, 32, 32),
    (1100, 1152, 192, 64, 64), (500, 3072, 64, 128, 64), (1000, 2048, 72, 32, 32), (1500, 3072, 40, 128, 128), (3900, 1152, 36, 0, 32),
    (7100, 1152, 24, 64, 64), (9000, 2080, 20, 160, 64), (17000, 1152, 16, 128, 128), (20000, 1184, 12, 32, 64),
])
def test_layer_equals_its_halves(M, K, N, r, g, schedule, asym, monkeypatch):
    print(f"[case] fields {schedule} asym={asym} M={M} K={K} N={N} r={r} g={g}", flush=True)
    monkeypatch.setenv("DIROTQ_W4A4_KERNEL", schedule)
    gen = torch.Generator(device="cuda").manual_seed(M + K + N)
    x = torch.randn(M, K, device="cuda", generator=gen).bfloat16()
    x[0] = 0.0                                             # groups of scale 0
    Qt = (torch.randn(K, K, device="cuda", generator=gen) / math.sqrt(K)).bfloat16()
    codes = torch.randint(-7, 8, (N, K - r), device="cuda", generator=gen, dtype=torch.int8)
    sw = (torch.rand(N, (K - r) // g, device="cuda", generator=gen) * 0.01 + 0.001).half()
    Wh = torch.randn(N, r, device="cuda", generator=gen).bfloat16() if r else None
    bias = torch.randn(N, device="cuda", generator=gen).bfloat16()
    blob = B.import_weights(Wh, codes, sw, N, K, r, g)
    if asym:
        y = B.linear_asym(x, Qt, blob, N, r, g, bias=bias)
        halves = B.rotate_quantize_asym(x, Qt, r, g)
        want = B.w4a4_gemm_asym(*halves, blob, M, N, K, r, g, bias=bias, out_dtype=torch.bfloat16)
    else:
        y = B.linear(x, Qt, blob, N, r, g, bias=bias)
        halves = B.rotate_quantize(x, Qt, r, g)
        want = B.w4a4_gemm(*halves, blob, M, N, K, r, g, bias=bias, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    assert torch.equal(y, want)


def test_shared_input_with_one_output_on_nibbles(monkeypatch):
    """Two outputs of one input: where one's kernel reads nibbles both do, and each equals its own layer."""
    monkeypatch.delenv("DIROTQ_W4A4_KERNEL", raising=False)
    gen = torch.Generator(device="cuda").manual_seed(5)
    M, K, r, g = 1000, 1152, 64, 64
    x = torch.randn(M, K, device="cuda", generator=gen).bfloat16()
    Qt = (torch.randn(K, K, device="cuda", generator=gen) / math.sqrt(K)).bfloat16()
    for Ns in ([64, 3072], [3072, 2048], [64, 96]):
        blobs = []
        for N in Ns:
            codes = torch.randint(-7, 8, (N, K - r), device="cuda", generator=gen, dtype=torch.int8)
            sw = (torch.rand(N, (K - r) // g, device="cuda", generator=gen) * 0.01 + 0.001).half()
            blobs.append(B.import_weights(torch.randn(N, r, device="cuda", generator=gen).bfloat16(), codes, sw, N, K, r, g))
        ys = B.linear_shared(x, Qt, blobs, Ns, r, g)
        for N, blob, y in zip(Ns, blobs, ys):
            assert torch.equal(y, B.linear(x, Qt, blob, N, r, g))

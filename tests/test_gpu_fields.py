"""Whole W4A4 layers whose kernel A hands the codes over in field form, against the two halves called on their own (nibbles): the
same codes, scales and sums in the same order, so the outputs are equal bit for bit.  Every form of kernel A on 256 CUs (few tokens:
always nibbles; K in two halves; 128 x 128 through registers and by copies; 128 x 160 and 128 x 256 by copies; several rounds of the
largest tiles; last stages of 32 channels) and every kernel B that reads the field form, all group sizes, split points inside a
tile, asymmetric codes (always nibbles), cut tiles, workgroups that walk several tiles.  The workspace shows which form the
codes had."""
import math

import pytest
import torch

from paper_2605_16732_amd import binding as B

pytestmark = pytest.mark.gpu


def _codes_in(workspace, M, K, r):
    """The x_l section of a layer's workspace (behind x_h, sections 256-byte aligned)."""
    at = (2 * M * r + 255) // 256 * 256
    return workspace[at:at + M * (K - r) // 2].view(M, (K - r) // 2)


@pytest.mark.parametrize("schedule,asym", [("tile", False), ("tile", True), ("large", False), ("small", False)])
@pytest.mark.parametrize("M,K,N,r,g,fields", [
    (1, 640, 96, 0, 64, False), (37, 640, 320, 64, 64, False), (70, 704, 136, 128, 64, False), (33, 1280, 100, 128, 128, False),
    (300, 672, 130, 32, 32, False), (1100, 1152, 192, 64, 64, False), (500, 3072, 64, 128, 64, True), (1000, 2048, 72, 32, 32, True),
    (2000, 1152, 200, 64, 64, True), (1000, 3072, 300, 128, 64, True), (1800, 2080, 52, 32, 32, True),
    (1500, 3072, 40, 128, 128, True), (3900, 1152, 36, 0, 32, True), (7100, 1152, 24, 64, 64, True), (9000, 2080, 20, 160, 64, True),
    (17000, 1152, 16, 128, 128, True), (20000, 1184, 12, 32, 64, True),
    (17000, 1152, 1030, 64, 64, True), (9000, 1184, 1100, 32, 32, True),     # more tiles than workgroups
])
def test_layer_equals_its_halves(M, K, N, r, g, fields, schedule, asym, monkeypatch):
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
    ws = torch.zeros(B.workspace_bytes(M, K, r, g), device="cuda", dtype=torch.uint8)
    if asym:
        y = B.linear_asym(x, Qt, blob, N, r, g, bias=bias, workspace=ws)
        halves = B.rotate_quantize_asym(x, Qt, r, g)
        want = B.w4a4_gemm_asym(*halves, blob, M, N, K, r, g, bias=bias, out_dtype=torch.bfloat16)
    else:
        y = B.linear(x, Qt, blob, N, r, g, bias=bias, workspace=ws)
        halves = B.rotate_quantize(x, Qt, r, g)
        want = B.w4a4_gemm(*halves, blob, M, N, K, r, g, bias=bias, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    assert torch.equal(y, want)
    assert torch.equal(_codes_in(ws, M, K, r), halves[1]) != (fields and not asym)


@pytest.mark.parametrize("Ns,fields", [([64, 1500], False), ([1500, 64], False), ([1500, 1400], True), ([64, 96], False)])
def test_shared_input_with_outputs_of_one_or_both_forms(Ns, fields, monkeypatch):
    """Two outputs of one input: the codes are in field form only where both outputs' kernels read it (1400 and 1500 channels: 128 x
    128 tiles; 64 and 96: the split-K kernel, which reads nibbles), and each output equals its own layer.  2000 tokens: kernel A
    is the 128 x 128 form, which writes what it is asked for."""
    monkeypatch.delenv("DIROTQ_W4A4_KERNEL", raising=False)
    print(f"[case] shared input, N={Ns}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(5)
    M, K, r, g = 2000, 1152, 64, 64
    x = torch.randn(M, K, device="cuda", generator=gen).bfloat16()
    Qt = (torch.randn(K, K, device="cuda", generator=gen) / math.sqrt(K)).bfloat16()
    blobs = []
    for N in Ns:
        codes = torch.randint(-7, 8, (N, K - r), device="cuda", generator=gen, dtype=torch.int8)
        sw = (torch.rand(N, (K - r) // g, device="cuda", generator=gen) * 0.01 + 0.001).half()
        blobs.append(B.import_weights(torch.randn(N, r, device="cuda", generator=gen).bfloat16(), codes, sw, N, K, r, g))
    ws = torch.zeros(B.workspace_bytes(M, K, r, g), device="cuda", dtype=torch.uint8)
    ys = B.linear_shared(x, Qt, blobs, Ns, r, g, workspace=ws)
    nibbles = B.rotate_quantize(x, Qt, r, g)[1]
    assert torch.equal(_codes_in(ws, M, K, r), nibbles) != fields
    for N, blob, y in zip(Ns, blobs, ys):
        assert torch.equal(y, B.linear(x, Qt, blob, N, r, g))

"""Short calls (few elements, rows of at most 256 key blocks) run the block statistics, the V tiles, the predictor and the
K quantization in two launches; larger calls run them one by one.  A head computed in a short call must come out as the
same head inside a call that is too large to be one, bit for bit: mask, output and counters.  Sizes at the edges of the
fused kernel: one and two key blocks, a workgroup's 8 rows, 64 / 128 / 129 / 256 key blocks, ragged ends."""
import pytest

pytestmark = pytest.mark.gpu

SHORT_MAX, SHORT_MAX_LONG_ROWS = 3 << 23, 1 << 24   # elements per tensor up to 128, up to 256 key blocks


@pytest.mark.parametrize("N,d,dtype,causal,kw", [
    (193, 128, "fp16", True, {}), (300, 64, "bf16", False, {}), (1024, 64, "fp16", False, {"pv_fp8": True}),
    (1100, 128, "bf16", True, {}), (4096, 128, "bf16", False, {"qk16": True}), (8192, 64, "bf16", True, {}),
    (8193, 128, "fp16", False, {}), (16384, 128, "bf16", False, {}), (16321, 64, "bf16", True, {"pv_fp8": True})])
def test_short_call_equals_the_same_heads_in_a_large_one(N, d, dtype, causal, kw):
    import torch
    import paper_2502_18137_amd as sp
    most = SHORT_MAX if (N + 63) // 64 <= 128 else SHORT_MAX_LONG_ROWS
    heads = most // (N * d) + 1
    H = min(heads, 128)
    B = -(-heads // H)
    print(f"B={B} H={H} N={N} d={d} {dtype} causal={causal} {kw}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + d)
    dt = torch.float16 if dtype == "fp16" else torch.bfloat16
    draw = lambda: torch.randn(B, H, (N + 127) // 128, d, generator=g, device="cuda").repeat_interleave(128, 2)[:, :, :N]
    Q, K, V = ((draw() + 0.4 * torch.randn(B, H, N, d, generator=g, device="cuda")).to(dt) for _ in range(3))
    K += 0.5                                                    # a mean for the quantization to take out
    args = dict(causal=causal, return_mask=True, return_stats=True, **kw)
    big = sp.sparge_forward(Q, K, V, 0.9, 0.6, -5.0, **args)
    big_mask = sp.sparge_predict(Q, K, 0.9, 0.6, causal=causal)
    for b, h in ((0, 0), (B - 1, H - 1)):
        one = tuple(t[b:b + 1, h:h + 1] for t in (Q, K, V))
        for x, y, what in zip(sp.sparge_forward(*one, 0.9, 0.6, -5.0, **args), big, ("output", "mask", "counters")):
            assert torch.equal(x, y[b:b + 1, h:h + 1]), (what, b, h)
        assert torch.equal(sp.sparge_predict(*one[:2], 0.9, 0.6, causal=causal), big_mask[b:b + 1, h:h + 1])
    assert 0 < int(big[1].sum()) and (N < 2000 or int(big[1].sum()) < big[1].numel())   # something is left out


@pytest.mark.parametrize("N,d,H", [(64, 64, 2), (1100, 128, 3), (20000, 64, 2)])
def test_quantization_does_not_depend_on_the_call_that_makes_it(N, d, H):
    """sparge_attn and sparge_quantize run the statistics without norms and self-similarity, sparge_forward with them:
    with every block kept the outputs are the same bits."""
    import torch
    import paper_2502_18137_amd as sp
    g = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V = (torch.randn(1, H, N, d, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    K += 0.5
    print(f"H={H} N={N} d={d}", flush=True)
    dense = sp.sparge_forward(Q, K, V, 1.0, 2.0, -5.0)          # theta above every similarity: all blocks kept
    assert torch.equal(sp.sparge_attn(Q, K, V, None, -5.0), dense)
    assert torch.equal(sp.sparge_attn_quantized(*sp.sparge_quantize(Q, K)[:4], V, None, -5.0), dense)

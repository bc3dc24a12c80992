"""Item counts around the number of resident workgroups (two per compute unit): up to it every workgroup computes the
one item at its own position and no counter is used, one item more and the counters start behind those positions; with
a few items per workgroup every workgroup draws from its own range first and from the other ranges once that is empty.
Each (batch, head) must come out as in a call of its own (whose few items never need a counter), bit for bit, and
the first and last ones as the oracle has them."""
import numpy as np
import pytest

from oracle import sparge_oracle as so
from tests.helpers import REF_SLACK, f32, small_workload, to_torch
from synth import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extra,d,causal", [(-1, 64, False), (0, 128, False), (1, 64, True), (9, 128, False), (1033, 64, False)])
def test_items_around_the_resident_workgroups(extra, d, causal):
    import torch
    import paper_2502_18137_amd as sp
    slots = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    n = slots + extra                       # items: n (batch, head) pairs of one Q block each
    H = next(h for h in range(128, 0, -1) if n % h == 0)
    B, N, lam = n // H, 70, -6.0
    print(f"{n} items: B={B} H={H} N={N} d={d} causal={causal}", flush=True)
    w = small_workload(f"items{extra}", N=N, d=d, dtype="bf16", H=n, causal=causal, seed=31, noise=1.0)
    x = make_workload(w)
    Q, K, V = (to_torch(x[t].reshape(B, H, N, d), "bf16") for t in "qkv")
    O, stats = sp.sparge_attn(Q, K, V, None, lam, causal=causal, return_stats=True)
    for b in range(B):                      # 4 heads a call
        for h0 in range(0, H, 4):
            one = tuple(t[b:b + 1, h0:h0 + 4] for t in (Q, K, V))
            assert torch.equal(sp.sparge_attn(*one, None, lam, causal=causal), O[b:b + 1, h0:h0 + 4]), (b, h0)
    assert (stats[..., 0] == stats[..., 2]).all() and (stats[..., 2] == 2).all()
    flat = O.reshape(n, N, d).float().cpu().numpy().astype(np.float64)
    for g in (0, n - 1):
        ref = so.sparse_attention(x["q"][0, g], x["k"][0, g], x["v"][0, g], None, lam=f32(lam), causal=causal,
                                  quant=True, pv_dtype="bf16", ref_slack=REF_SLACK)
        assert so.rel_l1(flat[g], so.round16(ref.O, "bf16")) <= 2e-3


@pytest.mark.parametrize("B,H", [(1, 1), (1, 64), (5, 13), (3, 127)])
def test_counters_are_set_whatever_they_held(B, H, monkeypatch):
    """The execution counters come in uninitialised and are set by an earlier kernel of the call: block statistics (short
    calls and others) or a kernel of its own, with a workgroup per 256 of them."""
    import torch
    import paper_2502_18137_amd as sp
    g = torch.Generator(device="cuda").manual_seed(H)
    Q, K, V = (torch.randn(B, H, 100, 64, generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    ops, tiles = sp.sparge_quantize(Q, K)[:4], sp.sparge_v_tiles(V)
    empty = torch.empty
    monkeypatch.setattr(torch, "empty", lambda *a, **k: empty(*a, **k).fill_(-1) if k.get("dtype") == torch.int64 else empty(*a, **k))
    want = torch.tensor([2, 8, 2, 8], device="cuda").expand(B, H, 4)     # one Q block of two key blocks, all executed
    inf = float("inf")
    tiled = torch.full((B, H, 4), -1, dtype=torch.int64, device="cuda")
    sp.sparge_attn_tiled(*ops, tiles, V, None, -inf, stats=tiled)
    for what, got in (("forward", sp.sparge_forward(Q, K, V, 1.0, 2.0, -inf, return_stats=True)[1]),
                      ("attn", sp.sparge_attn(Q, K, V, None, -inf, return_stats=True)[1]),
                      ("attn, 16-bit Q K^T", sp.sparge_attn(Q, K, V, None, -inf, return_stats=True, qk16=True)[1]),
                      ("attn_quantized", sp.sparge_attn_quantized(*ops, V, None, -inf, return_stats=True)[1]),
                      ("attn_tiled", tiled)):
        print(f"B={B} H={H} {what}", flush=True)
        assert torch.equal(got, want), what

"""Calls of few row groups run the flash loop with a workgroup per 32-row group whose waves share the group's tiles
(attn_split.hip); larger calls give a row group to one wave (attn.hip).  Both decide, round and add in the same order, so heads
in a call of their own must come out as the same heads of a call that is too large for the shared form, bit for bit:
output and execution counters.  Sizes at the edges of a row group, a key block, a round of four tiles, the longest list (as
many row groups as there are compute units in one head) and the causal lines beyond it; random masks with rows that keep
nothing, scores wide enough for the reference maximum to move and for the stage-2 test to skip; the few heads also lie token by
token in memory."""
import pytest

pytestmark = pytest.mark.gpu


def shared_form(heads, N, d, causal, qk16, units):
    """The line between the kernels (attn_split_pays), for the sizes below to lie on the side they are meant for."""
    Tn, groups = (N + 63) // 64, heads * ((N + 31) // 32)
    if Tn > 128 or groups <= units:
        return Tn <= 128
    if not causal or Tn > 64 or (qk16 and d == 128):
        return False
    return (8 * groups <= 9 * units and Tn >= 4 or 2 * groups <= 3 * units and Tn >= 8
            or groups <= 2 * units and (Tn >= 32 or Tn >= 16 and heads % 8 == 0))


def calls(causal, d, qk16, units):
    """-> (heads, N) of calls that run the shared form."""
    yield from ((1, N) for N in (1, 31, 33, 64, 65, 129, 256, 257, 700, 1100, 4173, 32 * units - 31, 32 * units))
    yield from ((3, 700), (units // 2, 60), (8, 4 * units))
    if causal and not (qk16 and d == 128):
        yield from ((units // 8 + 1, 250), (3 * units // 32, 509), (16, 4 * units), (8, 8 * units), (5, 3 * 32 * units // 8 + 1))


@pytest.mark.parametrize("kw", [{}, {"pv_fp8": True}, {"qk16": True}], ids=["int8", "fp8", "qk16"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (64, "fp16"), (128, "bf16"), (128, "fp16")])
def test_a_head_of_its_own_equals_the_head_of_a_large_call(d, dtype, causal, kw):
    import torch
    import paper_2502_18137_amd as sp
    dt = torch.float16 if dtype == "fp16" else torch.bfloat16
    units = torch.cuda.get_device_properties(0).multi_processor_count
    skipped = 0
    for few, N in calls(causal, d, "qk16" in kw, units):
        groups, Tm, Tn = (N + 31) // 32, (N + 127) // 128, (N + 63) // 64
        heads = max(2 * units // groups, few) + 1           # one more than the shared form takes, causal or not
        H = min(heads, 128)
        B = -(-heads // H)
        assert shared_form(few, N, d, causal, "qk16" in kw, units) and not shared_form(B * H, N, d, causal, "qk16" in kw, units)
        keep, lam = (1.0, -3.0) if N % 2 else (0.4, -1.5)
        print(f"B={B} H={H} few={few} N={N} d={d} {dtype} causal={causal} {kw}", flush=True)
        g = torch.Generator(device="cuda").manual_seed(N + d)
        wide = 1 + 1.5 * torch.randn(B, H, Tn, 1, generator=g, device="cuda").abs().repeat_interleave(64, 2)[:, :, :N]
        Q, K, V = ((torch.randn(B, H, N, d, generator=g, device="cuda") * wide).to(dt) for _ in range(3))
        mask = (torch.rand(B, H, Tm, Tn, generator=g, device="cuda") < keep).to(torch.uint8)
        mask[0, 0, Tm // 2] = 0                             # a Q block that keeps nothing
        args = dict(causal=causal, return_stats=True, **kw)
        O, stats = sp.sparge_attn(Q, K, V, mask, lam, **args)
        assert torch.isfinite(O.float()).all()
        skipped += int((stats[..., 3] - stats[..., 1]).sum())
        for b, h in {(0, 0), (B - 1, H - few)}:             # `few` heads from there on
            *qkv, m = (t[b:b + 1, h:h + few].contiguous() for t in (Q, K, V, mask))
            if N % 2:                                       # token by token
                qkv = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in qkv]
            o, st = sp.sparge_attn(*qkv, m, lam, **args)
            assert torch.equal(o, O[b:b + 1, h:h + few]), (few, N, b, h)
            assert torch.equal(st, stats[b:b + 1, h:h + few]), (few, N, b, h)
    assert skipped > 0


def not_finite(kind, Q, K, V, N):
    """The kinds of infinities and NaN that scores, their maxima and P~ can meet (Q, K, V changed in place)."""
    inf, nan = float("inf"), float("nan")
    if kind == "K has infinities":
        K[:, :, 3, 5], K[:, :, N // 2, 5], K[:, :, N - 1, 9] = inf, -inf, inf
    elif kind == "NaN":
        K[:, :, N // 3, 7] = Q[:, :, N // 2, 2] = V[:, :, N - 1, 3] = nan
    elif kind == "a key block of NaN":
        K[:, :, :64] = nan
    elif kind == "Q rows of infinite scores":
        Q[:, :, ::37, 2] = inf
    elif kind == "all scores infinite":
        Q[..., 2] = inf
    elif kind == "first key blocks at -inf":
        Q[..., 1] = Q[..., 1].abs() + 0.5
        K[:, :, :200, 1] = -inf
    elif kind == "infinite V":
        V[:, :, 5, 3], V[:, :, N // 2, 4] = inf, -inf


@pytest.mark.parametrize("kw", [{}, {"pv_fp8": True}, {"qk16": True}], ids=["int8", "fp8", "qk16"])
@pytest.mark.parametrize("kind", ["K has infinities", "NaN", "a key block of NaN", "Q rows of infinite scores", "all scores infinite",
                                  "first key blocks at -inf", "infinite V"])
def test_infinities_and_nan_come_out_the_same(kind, kw):
    import torch
    import paper_2502_18137_amd as sp
    units = torch.cuda.get_device_properties(0).multi_processor_count
    for N, d, dt in ((100, 64, torch.bfloat16), (333, 128, torch.float16), (1100, 64, torch.float16), (1100, 128, torch.bfloat16)):
        groups, Tm, Tn = (N + 31) // 32, (N + 127) // 128, (N + 63) // 64
        H = min(2 * units // groups + 1, 128)
        B = -(-(2 * units // groups + 1) // H)
        g = torch.Generator(device="cuda").manual_seed(N + d)
        Q, K, V = (torch.randn(B, H, N, d, generator=g, device="cuda").to(dt) for _ in range(3))
        not_finite(kind, Q, K, V, N)
        masks = (None, (torch.rand(B, H, Tm, Tn, generator=g, device="cuda") < 0.6).to(torch.uint8))
        for causal in (False, True):
            for mask in masks:
                print(f"{kind}: B={B} H={H} N={N} d={d} {dt} causal={causal} mask={mask is not None} {kw}", flush=True)
                args = dict(causal=causal, return_stats=True, **kw)
                O, stats = sp.sparge_attn(Q, K, V, mask, -3.0, **args)
                one = [t[:1, :1].contiguous() for t in (Q, K, V)]
                o, st = sp.sparge_attn(*one, None if mask is None else mask[:1, :1].contiguous(), -3.0, **args)
                assert torch.equal(st, stats[:1, :1])
                same = (o == O[:1, :1]) | (o.isnan() & O[:1, :1].isnan())
                assert same.all(), (kind, N, d, causal, int((~same).sum()))

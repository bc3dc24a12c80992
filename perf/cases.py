"""The work a user of this framework has it do, as timed cases.

A case is a dict of plain values.  `listed()` holds the named ones, `draw(rng)` gives further cases of the same
ranges; `prepare` makes what a program has in hand before the call (tensors on the GPU, per-head settings, the
workspace and the output it keeps), `run` makes one pass through the public entry points.

Inputs follow the recipes of synth/workloads.py, drawn on the GPU: smooth random fields on a (t, h, w) grid along
a Hilbert curve for visual tokens, segments that share a centroid for short mixed prompts, low-rank drift with a
sink and periodic position components for causal language.  V is white noise.
"""
import math

import torch

import paper_2502_18137_amd as sp

DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16}

# op: forward = the whole of Algorithm 1; visual = Hilbert permutation of Q, K, V, the forward pass and the inverse
# permutation of O (Sec. 3.7); predict = block mask and its index lists, for callers with their own kernels;
# masked = quantized attention under a block mask of the caller's; tune = hyper-parameter search of one layer.
# keep: the program holds one workspace and one output for all its calls (a serving loop); otherwise they come from
# torch's allocator on each call.  kept: share of the blocks that such inputs keep, for work() alone.
BASE = dict(op="forward", B=1, H=2, N=0, d=64, dtype="bf16", causal=False, inputs="segments", T=1, h=0, w=0, text=0,
            st=1.0, ss=1.0, noise=0.3, tau=0.9, theta=0.5, lam=-5.0, layout="bhnd", pv_fp8=False, qk16=False,
            keep=True, kept=1.0)


def _case(**kw):
    c = dict(BASE, **kw)
    if c["inputs"] == "field":
        c["N"] = c["text"] + c["T"] * c["h"] * c["w"]
    return c


def listed():
    return [
        # The smallest calls: one layer of a small model on 2048 tokens (the "tiny" configuration), and a short
        # ragged causal prompt in the layout a projection leaves behind.  Launches and latency count here.
        _case(name="tiny", H=2, N=2048, d=64, dtype="fp16", theta=0.6, kept=0.65),
        _case(name="short_prompt", H=8, N=1100, d=128, causal=True, tau=0.8, lam=-4.0, layout="bnhd", keep=False, kept=0.6),
        # A batch of small images, odd token count, fp16.
        _case(name="image_batch", B=4, H=16, d=64, dtype="fp16", inputs="field", h=33, w=32, ss=4.0, noise=0.2, tau=0.95,
              lam=-8.0, layout="bnhd", kept=0.93),
        # One 64 x 64 image with its text tokens in front: permuted, attended, put back.
        _case(name="image_joint", op="visual", H=24, d=128, inputs="field", h=64, w=64, text=77, ss=6.0, noise=0.2, tau=0.95,
              lam=-8.0, kept=0.85),
        # The video and long-video configurations, the headline work; and a long one with the FP8 P~V product.
        _case(name="video", H=48, d=64, inputs="field", T=13, h=30, w=45, st=2.0, ss=5.0, noise=0.2, lam=-6.0, kept=0.73),
        _case(name="video_fp8", H=24, d=128, inputs="field", T=29, h=24, w=32, st=3.0, ss=6.0, noise=0.15, pv_fp8=True,
              kept=0.7),
        _case(name="longvideo", H=24, d=128, inputs="field", T=20, h=48, w=48, st=3.0, ss=8.0, noise=0.15, kept=0.69),
        # Causal language prefill at the configuration's length, and a shorter one with the unquantized Q K^T.
        _case(name="language", H=32, N=32768, d=128, causal=True, inputs="language", tau=0.95, theta=0.6, lam=-10.0,
              kept=0.42),
        _case(name="language_qk16", H=32, N=8192, d=128, causal=True, inputs="language", tau=0.95, theta=0.6, lam=-10.0,
              qk16=True, keep=False, kept=0.46),
        # The predictor alone on 64k tokens, its mask as index lists (the predictor-overhead table's shape).
        _case(name="predict_64k", op="predict", H=32, N=65536, d=128, inputs="language", kept=0.5),
        # Attention under a given mask of half the blocks (the shape of the speed-against-sparsity figure).
        _case(name="masked_half", op="masked", H=24, N=22272, d=128, lam=-math.inf, kept=0.5),
        # The per-head search over a small grid on two inputs of one layer.
        _case(name="tune", op="tune", H=4, N=1536, d=64, dtype="fp16", keep=False, kept=0.8),
    ]


def _loguniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any op, any shape up to the largest listed one's cost."""
    op = rng.choice(["forward"] * 6 + ["visual"] * 2 + ["masked"] * 2 + ["predict", "tune"])
    c = dict(BASE, op=op, d=rng.choice([64, 128]), dtype=rng.choice(["bf16", "bf16", "fp16"]),
             layout=rng.choice(["bhnd", "bhnd", "bnhd"]), keep=rng.random() < 0.6, tau=rng.choice([0.8, 0.9, 0.95]),
             theta=rng.choice([0.5, 0.6]), lam=rng.choice([-4.0, -5.0, -6.0, -8.0, -10.0]))
    inputs = "field" if op == "visual" else rng.choice(["segments", "field", "field", "language"])
    c["inputs"] = inputs
    if op == "tune":
        c.update(inputs="segments", H=rng.choice([2, 4]), N=_loguniform(rng, 500, 2500), keep=False, layout="bhnd")
        return c
    if inputs == "field":
        still = rng.random() < 0.4
        c.update(T=1 if still else rng.randint(5, 20), h=rng.randint(12, 64) if still else rng.randint(16, 48),
                 noise=rng.choice([0.15, 0.2]), st=rng.uniform(2, 3), text=rng.choice([0, 0, 77, rng.randint(1, 256)]))
        c.update(w=max(8, min(64, int(c["h"] * rng.uniform(0.7, 1.4)))))
        c.update(ss=rng.uniform(0.1, 0.17) * min(c["h"], c["w"]), kept=0.75)
        c["N"] = c["text"] + c["T"] * c["h"] * c["w"]
    else:
        c["N"] = _loguniform(rng, 300, 65536 if op == "predict" else 46080)
        c["causal"] = op != "masked" and (inputs == "language" or rng.random() < 0.4)
        c["kept"] = 0.8
    if op == "masked":
        c["kept"] = rng.choice([0.2, 0.4, 0.6, 0.8, 1.0])
        c["lam"] = rng.choice([-math.inf, -6.0])
    if op in ("forward", "masked"):
        variant = rng.choice(["int8"] * 4 + ["pv_fp8", "qk16"])
        c["pv_fp8"], c["qk16"] = variant == "pv_fp8", variant == "qk16"
    c["B"] = rng.choice([1, 1, 1, 2, 3]) if c["N"] < 6000 else 1
    c["H"] = rng.choice([2, 4, 8, 12, 16, 24, 32, 40, 48])
    most = max(work(x)["flops"] for x in listed()) * 0.8
    while c["H"] > 1 and (work(dict(c, kept=1.0))["flops"] > most or c["B"] * c["H"] * c["N"] * c["d"] > 4e8):
        c["H"] = max(1, c["H"] // 2)
    return c


# ---- inputs --------------------------------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + salt * 7919 + 17) % (1 << 62))
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda")


def _smoother(n, std):
    """[n, n]: periodic Gaussian average along an axis, rows of unit norm (unit variance in, unit variance out)."""
    i = torch.arange(n, device="cuda", dtype=torch.float32)
    dist = (i[:, None] - i[None, :]).abs()
    m = torch.exp(-0.5 * (torch.minimum(dist, n - dist) / std) ** 2)
    return m / m.norm(dim=1, keepdim=True)


def _field(c, g):
    """[B, H, N, d]: per channel a smooth field over the grid, in row-major grid order behind the text tokens."""
    B, H, d, T, h, w = (c[k] for k in ("B", "H", "d", "T", "h", "w"))
    x = _randn(g, B * H * d, T, h, w)
    x = x @ _smoother(w, c["ss"]).T
    x = _smoother(h, c["ss"]) @ x
    if T > 1:
        x = (_smoother(T, c["st"]) @ x.reshape(B * H * d, T, h * w)).reshape(B * H * d, T, h, w)
    x = x.reshape(B, H, d, T * h * w).transpose(2, 3)
    x = x + c["noise"] * _randn(g, *x.shape)
    return x if not c["text"] else torch.cat([_randn(g, B, H, c["text"], d), x], dim=2)


def _segments(c, g):
    centroids = _randn(g, c["B"], c["H"], (c["N"] + 127) // 128, c["d"])
    x = centroids.repeat_interleave(128, dim=2)[:, :, :c["N"]]
    return x + c["noise"] * _randn(g, *x.shape)


def _language(c, gs):
    """Q and K [B, H, N, d]: noise + a slowly drifting low-rank component + periodic position components, both
    shared, + a sink in K's first token; the first 64 tokens carry nothing shared."""
    B, H, N, d = (c[k] for k in ("B", "H", "N", "d"))
    r, BH = 8, B * H
    basis = torch.linalg.qr(_randn(gs, BH, d, 3 * r))[0]                     # [BH, d, 3r], orthonormal columns
    u0 = _randn(gs, BH, d)
    u0 = u0 / u0.norm(dim=1, keepdim=True)
    t = torch.arange(N, device="cuda", dtype=torch.float64)
    rho = math.exp(-1 / 4096.0)                                             # correlation length of the drift
    eps = _randn(gs, BH, N, r).double()
    eps[:, 0] /= math.sqrt(1 - rho * rho)
    z = (math.sqrt(1 - rho * rho) * (eps * rho ** -t[:, None]).cumsum(1) * rho ** t[:, None]).float()
    ang = (2 * math.pi * t[:, None] / (512.0 * 2.0 ** torch.arange(r, device="cuda", dtype=torch.float64))).float()
    pos = torch.cat([torch.cos(ang), torch.sin(ang)], 1) / math.sqrt(r)     # [N, 2r]
    mix = torch.cat([6.0 * z, (4.0 * pos).expand(BH, N, 2 * r)], 2)         # [BH, N, 3r]
    shared = mix @ basis.transpose(1, 2).contiguous()
    shared[:, :64] = 0
    q = shared + _randn(gs, BH, N, d) + u0[:, None]
    k = shared + _randn(gs, BH, N, d)
    k[:, 0] = 4.0 * k.norm(dim=2).mean(1, keepdim=True) * u0
    return q.reshape(B, H, N, d), k.reshape(B, H, N, d)


def _lay(x, c):
    """The values in the case's 16-bit type and memory layout, as a [B, H, N, d] view."""
    x = x.to(DTYPES[c["dtype"]])
    return x.transpose(1, 2).contiguous().transpose(1, 2) if c["layout"] == "bnhd" else x.contiguous()


def _qkv(c, seed):
    if c["inputs"] == "language":
        q, k = _language(c, _gen(seed, 1))
    else:
        make = _field if c["inputs"] == "field" else _segments
        q, k = make(c, _gen(seed, 1)), make(c, _gen(seed, 2))
        if c["inputs"] == "field" and c["op"] != "visual":                  # tokens already along the curve
            perm = sp.sparge_hilbert_order(c["T"], c["h"], c["w"]).to("cuda").long() + c["text"]
            at = torch.cat([torch.arange(c["text"], device="cuda"), perm])
            q, k = q[:, :, at], k[:, :, at]
    q, k = _lay(q, c), _lay(k, c)
    return q, k, _lay(_randn(_gen(seed, 3), c["B"], c["H"], c["N"], c["d"]), c)


def prepare(case, seed):
    c = dict(BASE, **case)
    s = {"case": c}
    if c["op"] == "tune":
        s["inputs"] = [_qkv(c, 2 * seed + n + 1) for n in range(2)]
        return s
    s["Q"], s["K"], s["V"] = _qkv(c, seed)
    if c["op"] == "predict":
        del s["V"]
    H, like = c["H"], s["Q"]
    # per-head settings, as a search leaves them: around the case's values
    s["tau"] = [min(1.0, c["tau"] + 0.01 * ((h % 3) - 1)) for h in range(H)]
    s["theta"] = [c["theta"]] * H
    s["lam"] = [c["lam"] - 0.5 * (h % 2) for h in range(H)]
    if c["op"] == "visual":
        s["perm"] = sp.sparge_hilbert_order(c["T"], c["h"], c["w"]).to("cuda")
    if c["op"] == "masked":
        Tm, Tn = (c["N"] + 127) // 128, (c["N"] + 63) // 64
        m = torch.rand(c["B"], H, Tm, Tn, generator=_gen(seed, 4), device="cuda") < c["kept"]
        m[..., 0] = True
        s["mask"] = m.to(torch.uint8)
    s["ws"] = s["out"] = None
    if c["keep"] and c["op"] != "predict":
        entry = sp.WS_ATTN if c["op"] == "masked" else sp.WS_FORWARD
        s["ws"] = torch.empty(sp.sparge_workspace_bytes(like, entry, c["pv_fp8"]), dtype=torch.uint8, device="cuda")
        s["out"] = torch.empty_like(like)
    elif c["keep"]:
        s["ws"] = torch.empty(sp.sparge_workspace_bytes(like, sp.WS_PREDICT), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    c, op = s["case"], s["case"]["op"]
    if op == "forward":
        return sp.sparge_forward(s["Q"], s["K"], s["V"], s["tau"], s["theta"], s["lam"], causal=c["causal"], ws=s["ws"],
                                 out=s["out"], pv_fp8=c["pv_fp8"], qk16=c["qk16"])
    if op == "visual":
        q, k, v = (sp.sparge_permute_tokens(s[t], s["perm"], offset=c["text"]) for t in "QKV")
        o = sp.sparge_forward(q, k, v, s["tau"], s["theta"], s["lam"], causal=c["causal"], ws=s["ws"], out=s["out"])
        return sp.sparge_permute_tokens(o, s["perm"], offset=c["text"], inverse=True)
    if op == "predict":
        mask = sp.sparge_predict(s["Q"], s["K"], s["tau"], s["theta"], causal=c["causal"], ws=s["ws"])
        lut, count = sp.sparge_mask_to_lut(mask, s["Q"])
        return {"mask": mask, "lut": lut, "count": count}
    if op == "masked":
        o, stats = sp.sparge_attn(s["Q"], s["K"], s["V"], s["mask"], s["lam"], causal=c["causal"], return_stats=True,
                                  ws=s["ws"], out=s["out"], pv_fp8=c["pv_fp8"], qk16=c["qk16"])
        return {"O": o, "stats": stats}
    return sp.sparge_tune(s["inputs"], [0.7, 0.9], [0.3, 0.6], [-4.0, -8.0], 0.2, 0.21, causal=c["causal"])


def work(case):
    """Bytes: Q, K, V read once and O (the mask and its lists) written once.  flops: the two products on the kept
    blocks, counted at the 16-bit rate: an 8-bit product counts half."""
    c = dict(BASE, **case)
    elems = c["B"] * c["H"] * c["N"] * c["d"]
    full = 2.0 * c["B"] * c["H"] * c["N"] * c["N"] * c["d"] * (0.5 if c["causal"] else 1.0)
    if c["op"] == "predict":
        rows = c["B"] * c["H"] * math.ceil(c["N"] / 128)
        # the pooled product is in fp64, whose matrix rate is a thirty-second of the 16-bit one
        return {"bytes": 4.0 * elems + rows * (math.ceil(c["N"] / 64) * 5.0 + 4.0), "flops": full / (128 * 64) * 32}
    flops = full * c["kept"] * ((1.0 if c["qk16"] else 0.5) + (0.5 if c["pv_fp8"] else 1.0))
    if c["op"] == "tune":
        return {"bytes": 2 * 6.0 * elems, "flops": 2 * 7 * flops}  # per input: the full attention and six settings
    if c["op"] == "visual":
        return {"bytes": 8.0 * elems, "flops": flops}
    return {"bytes": 8.0 * elems, "flops": flops}


def tolerance(case):
    """With u the unit roundoff of the 16-bit type (2^-8 bf16, 2^-11 fp16), correct evaluations differ by independent
    roundings of P~ and O: relative 2-norm 0.6 u, and at most 0.015 (bf16) or 0.0014 (fp16) of a value or of the rms,
    both measured against fp64 attention on the same blocks and quantized operands; about four times that is stated.
    FP8 P~: 3.8e-2 and 0.22 against exact P~, and less between two that round it alike.  Whole values (masks, lists,
    counters) may differ where a statistic sits on its threshold."""
    c = dict(BASE, **case)
    if c["op"] == "predict":
        return {"rel": 0.0, "differ": 1e-4}
    if c["pv_fp8"]:
        return {"rel": 3e-2, "max": 0.9, "differ": 5e-3}
    if c["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.06, "differ": 5e-3}
    return {"rel": 1.2e-3, "max": 6e-3, "differ": 5e-3}

"""TopCdf of a row finds the cut in the ranking by bracketing it instead of sorting the row.  Rows of every kind the bracket
meets -- flat, peaked, equal entries (ties rank by ascending index) few and many, among others above and below them, one block with
all the mass, entries that underflow to 0, tau = 1 -- at the edges of the entries per lane and of the candidate count, against a
sorted row in fp64; and the time of rows with many equal entries beside that of others."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BLOCKS = [1, 2, 31, 32, 33, 64, 65, 127, 129, 256, 257, 513, 1025, 2048]


def sorted_rows(logits, tau):
    """-> kept by the sorted definition, and where the mass before an entry is too close to the threshold to say."""
    p = np.exp(logits - logits.max(axis=1, keepdims=True))
    p /= p.sum(axis=1, keepdims=True)
    order = np.argsort(-p, axis=1, kind="stable")
    ranked = np.take_along_axis(p, order, 1)
    before = np.cumsum(ranked, axis=1) - ranked
    kept, open_ = np.zeros(p.shape, bool), np.zeros(p.shape, bool)
    np.put_along_axis(kept, order, (before < tau) & (ranked > 0), 1)
    np.put_along_axis(open_, order, np.abs(before - tau) < 1e-9, 1)
    return kept, open_


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("kind", ["flat", "peaked", "wide", "steps", "half", "two", "most"])
def test_rows_against_the_sorted_definition(kind, causal):
    import torch
    import paper_2502_18137_amd as sp
    d = 64
    for n in BLOCKS:
        N = 64 * n
        g = torch.Generator(device="cuda").manual_seed(n)
        scale = {"flat": 0.05, "wide": 12.0, "half": 0.3, "most": 0.1}.get(kind, 1.0)
        K = torch.randn(1, 1, n, d, generator=g, device="cuda") * scale
        src = np.arange(n)                                   # block j is a copy of block src[j]
        if kind == "steps":                                  # runs of seven blocks with the same logit
            src = src // 7 * 7
        elif kind == "two":                                  # two values
            src = src % 2
        elif kind in ("half", "most"):                       # every second block (nine of ten) alike
            src = np.where(src % 2 == 0 if kind == "half" else src % 10 != 3, 0, src)
        K = K[:, :, torch.from_numpy(src).cuda()]
        K = K.repeat_interleave(64, 2).to(torch.bfloat16).contiguous()
        Q = torch.randn(1, 1, (n + 1) // 2, d, generator=g, device="cuda").repeat_interleave(128, 2)[:, :, :N]
        Q = torch.empty_like(K).copy_(Q)
        Tm = (N + 127) // 128
        q = torch.stack([Q[0, 0, 128 * i:128 * i + 128].double().mean(0) for i in range(Tm)]).cpu().numpy()
        k = K[0, 0].double().reshape(n, 64, d).mean(1).cpu().numpy()
        logits = q @ k.T / 8.0
        logits = logits[:, src]                              # equal blocks: the same bits, whatever the product's order
        for tau in (1e-3, 0.5, 0.9, float(np.float32(0.999))):
            mask = sp.sparge_predict(Q, K, tau, -2.0, causal=causal).cpu().numpy()[0, 0].astype(bool)
            t = float(np.float32(tau))
            for i in range(Tm):
                seen = min(n, 2 * i + 2) if causal else n
                kept, open_ = sorted_rows(logits[i:i + 1, :seen], t)
                want = kept[0].copy()
                if causal:
                    want[min(2 * i, seen - 1)] = True
                wrong = (mask[i, :seen] != want) & ~open_[0]
                assert not wrong.any(), (kind, n, tau, i, np.flatnonzero(wrong)[:5])
                assert not mask[i, seen:].any()


@pytest.mark.parametrize("n", BLOCKS)
def test_equal_entries_rank_by_index_and_one_entry_can_hold_everything(n):
    import torch
    import paper_2502_18137_amd as sp
    Q = torch.ones(1, 1, 64 * n, 64, device="cuda", dtype=torch.bfloat16)
    K = torch.ones_like(Q)
    print(n, flush=True)
    for tau in (0.3, 0.7, 1.0):
        mask = sp.sparge_predict(Q, K, tau, -2.0).cpu().numpy()[0, 0]
        t = float(np.float32(tau)) * n
        if abs(t - round(t)) > 1e-6 * n or tau == 1.0:       # (a cut on the threshold is anybody's; tau = 1 has none there)
            want = np.arange(n) < np.ceil(t)
            assert (mask == want).all(), tau
    K[:, :, 64 * (n // 2):64 * (n // 2) + 64] = 2000.0       # everything else underflows to 0
    for tau in (0.3, 1.0):
        mask = sp.sparge_predict(Q, K, tau, -2.0).cpu().numpy()[0, 0]
        assert (mask == (np.arange(n) == n // 2)).all(), tau


def test_rows_of_equal_entries_take_no_longer():
    """Rows whose cut lies among many equal entries (repeated or padded tokens): the predictor call takes at most a fifth longer
    than on ordinary ones (a bracket that only halves needs 50 probes there and took 1.4 times as long)."""
    import torch
    import paper_2502_18137_amd as sp
    H, N, d = 48, 17550, 64
    Tn = (N + 63) // 64
    g = torch.Generator(device="cuda").manual_seed(1)
    Q = torch.randn(1, H, (N + 127) // 128, d, generator=g, device="cuda").repeat_interleave(128, 2)[:, :, :N].to(torch.bfloat16).contiguous()
    K = torch.randn(1, H, Tn, d, generator=g, device="cuda")
    alike = {"ordinary": torch.arange(Tn), "constant": torch.zeros(Tn, dtype=torch.long),
             "half": torch.where(torch.arange(Tn) % 2 == 0, 0, torch.arange(Tn)), "padded": torch.arange(Tn).clamp(max=Tn * 6 // 10)}
    keys = {k: K[:, :, src.cuda()].repeat_interleave(64, 2)[:, :, :N].to(torch.bfloat16).contiguous() for k, src in alike.items()}
    ws = torch.empty(sp.sparge_workspace_bytes(Q, sp.WS_PREDICT), dtype=torch.uint8, device="cuda")
    times = {k: [] for k in keys}
    for _ in range(9):
        for k, x in keys.items():
            sp.sparge_predict(Q, x, 0.9, -2.0, ws=ws)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                sp.sparge_predict(Q, x, 0.9, -2.0, ws=ws)
            b.record()
            torch.cuda.synchronize()
            times[k].append(a.elapsed_time(b) * 100)    # us a call
    us = {k: sorted(t)[4] for k, t in times.items()}
    print({k: round(t, 1) for k, t in us.items()}, flush=True)
    assert max(us.values()) <= 1.2 * us["ordinary"]

"""The output of the flash loop by its bits: every product, maximum and sum of it has one order (P~ enters the row sum l one
after the other, tile by tile), so that the bits of a call are a property of the library that no change of speed may move.
Recorded here as SHA-256 of the 16-bit output for fixed inputs, on both kernels (calls of few row groups and the others),
causal or not, and in the three product variants; scores are wide enough for the reference maximum to move, and lambda
skips products."""
import hashlib

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = {   # B, H, N, d, dtype, causal, variant -> the digest's first 16 digits
    (1, 2, 2048, 64, "fp16", False, "int8"): "5dcff88fefb9aebb",
    (1, 8, 1100, 128, "bf16", True, "int8"): "e3fab528b18a8df7",
    (1, 3, 777, 128, "fp16", False, "fp8"): "e9204e2c553faf2d",
    (1, 1, 5000, 64, "bf16", True, "fp8"): "25d9ff25ea1fc46d",
    (1, 2, 1400, 128, "bf16", False, "qk16"): "01d32539a9ca7230",
    (1, 24, 3000, 64, "bf16", False, "int8"): "949012d0d9bde376",
    (1, 12, 5000, 128, "fp16", True, "int8"): "bdbac08948b7d88b",
    (2, 8, 4173, 128, "bf16", False, "int8"): "b71ff466a49e1a23",
    (1, 20, 2500, 64, "fp16", True, "fp8"): "5b4eda1685d4d3b2",
    (1, 16, 3333, 128, "bf16", True, "qk16"): "17120bd82546467d",
}


@pytest.mark.parametrize("case", list(CASES), ids=lambda c: "-".join(map(str, c)))
def test_output_bits(case):
    import torch
    import paper_2502_18137_amd as sp
    B, H, N, d, dtype, causal, variant = case
    r = np.random.Generator(np.random.Philox(N + d))
    Tm, Tn = (N + 127) // 128, (N + 63) // 64
    wide = np.repeat(1 + 1.5 * np.abs(r.standard_normal((B, H, Tn, 1), np.float32)), 64, axis=2)[:, :, :N]
    dt = torch.float16 if dtype == "fp16" else torch.bfloat16
    Q, K, V = (torch.from_numpy(r.standard_normal((B, H, N, d), np.float32) * wide).to(dt).cuda() for _ in range(3))
    mask = torch.from_numpy((r.random((B, H, Tm, Tn)) < 0.6).astype(np.uint8)).cuda()
    lam = [-6.0 + 0.25 * (h % 3) for h in range(H)]
    O = sp.sparge_attn(Q, K, V, mask, lam, causal=causal, pv_fp8=variant == "fp8", qk16=variant == "qk16")
    got = hashlib.sha256(O.contiguous().view(torch.int16).cpu().numpy().tobytes()).hexdigest()[:16]
    print(f"    {case}: \"{got}\",", flush=True)
    assert got == CASES[case]

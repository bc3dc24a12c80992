"""Causal rows of up to 2048 key blocks rank only the key blocks they see, with a quarter, half or all of the ranks a full row
takes; longer rows are sorted in LDS with all their ranks, the unseen ones masked.  Logits that no row sees are not computed in
either.  Sequence lengths whose rows cross every one of these edges (ranks per lane 4 and less, 8, 16, 32, and the rows
sorted in LDS), ragged ends, workspaces filled with NaN: the mask against the oracle."""
import pytest

from oracle import sparge_oracle as so
from tests.helpers import f32, gpu_inputs, small_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("key_blocks,d", [(5, 64), (130, 128), (250, 64), (301, 64), (512, 128), (641, 64), (1100, 64), (2051, 64)])
def test_causal_rows_against_the_oracle(key_blocks, d):
    import torch
    import paper_2502_18137_amd as sp
    N = key_blocks * 64 - 23
    w = small_workload(f"rows{key_blocks}", N=N, d=d, dtype="bf16", H=1, causal=True, seed=key_blocks, noise=0.6)
    print(f"{key_blocks} key blocks, N={N} d={d}", flush=True)
    x, Q, K, _ = gpu_inputs(w)
    ws = torch.empty(sp.sparge_workspace_bytes(Q, sp.WS_PREDICT), dtype=torch.uint8, device="cuda").fill_(255)   # NaN
    mask = sp.sparge_predict(Q, K, w.tau, w.theta, causal=True, ws=ws).cpu().numpy()
    pr = so.predict(x["q"][0, 0], x["k"][0, 0], f32(w.tau), f32(w.theta), causal=True)
    assert not ((mask[0, 0] != pr.mask) & ~pr.dont_care).any()
    assert pr.dont_care.mean() < 0.05

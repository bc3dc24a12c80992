"""The workgroups of the K statistics take their blocks in an order of their own: an eighth of a head per XCD, and across
heads where a head has fewer than 16 blocks.  Every block must be taken once and written to its own place: self-similarity
per block and token mean per head against fp64, at block counts on both sides of 16 and of multiples of 8, with numbers of
blocks that are no multiple of 128, in short calls and in others, in both memory layouts."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("key_blocks,heads,d", [(1, 37, 64), (1, 6200, 64), (3, 50, 128), (4, 1031, 128), (15, 19, 64), (15, 229, 128),
                                                (16, 3, 64), (16, 400, 64), (17, 5, 128), (23, 290, 64), (31, 2, 64), (258, 3, 64)])
def test_every_k_block_is_taken_once(key_blocks, heads, d):
    import torch
    import paper_2502_18137_amd as sp
    N, H = key_blocks * 64 - 11, next(h for h in range(128, 0, -1) if heads % h == 0)
    B = heads // H
    print(f"{key_blocks} key blocks, B={B} H={H} N={N} d={d}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(key_blocks * 7 + d)
    level = torch.rand(B, H, key_blocks, 1, generator=g, device="cuda").repeat_interleave(64, 2)[:, :, :N]
    K = (torch.randn(B, H, N, d, generator=g, device="cuda") + 3 * level).to(torch.bfloat16)      # every block its own similarity
    if heads % 2:
        K = K.transpose(1, 2).contiguous().transpose(1, 2)
    _, _, sim = sp.sparge_predict(K, K, 0.9, 0.5, return_sims=True)
    mean = sp.sparge_quantize(K, K)[4]
    x = K.double()
    pad = torch.cat([x / x.norm(dim=3, keepdim=True), x.new_zeros(B, H, 11, d)], 2).reshape(B, H, key_blocks, 64, d)
    rows = torch.full((key_blocks,), 64.0, dtype=torch.float64, device="cuda")
    rows[-1] = 64 - 11
    want = (pad.sum(3) / rows[:, None]).pow(2).sum(3)
    assert torch.allclose(sim, want, rtol=1e-12, atol=0)        # fp64 sums of 64 x d terms in another order
    assert torch.allclose(mean.double(), x.mean(2), rtol=2.0 ** -23, atol=1e-12)

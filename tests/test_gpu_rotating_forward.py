"""The forward of a few rows that rotates its chunk inside the attention launch, against the same call behind the
rotation pre-pass (taken where the chunk keys are not 16-byte aligned): bit-identical outputs and staged operands,
at the edges of its tiles, tables and frames."""
import pytest

import workloads as wl
from helpers import dev_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,pairs,gh,gw,B,H,group,C,Fc,bf,resident", [
    (64, (12, 10, 10), 1, 1, 1, 1, 1, 3, 1, 0, 0),       # one token
    (64, (12, 10, 10), 3, 11, 2, 3, 1, 4, 3, 1, 2),      # 33-token frames, causal, one row past a tile
    (64, (12, 10, 10), 8, 16, 1, 2, 1, 6, 3, 0, 6),      # eight waves, twelve full chunk tiles
    (64, (12, 10, 10), 8, 16, 2, 12, 1, 4, 3, 0, 2),     # four waves, twelve: the most that they rotate
    (64, (12, 10, 10), 16, 20, 1, 2, 1, 4, 2, 0, 4),     # eight waves, twenty chunk tiles, a full table
    (64, (0, 16, 16), 4, 8, 1, 2, 1, 3, 2, 0, 3),        # no temporal pairs
    (128, (22, 21, 21), 2, 3, 2, 2, 3, 40, 40, 0, 7),    # many frames to a tile, candidates, 985 entries: staged after all
    (128, (22, 21, 21), 2, 3, 2, 2, 3, 35, 35, 0, 7),    # 875 entries
    (128, (64, 0, 0), 5, 13, 1, 3, 1, 3, 2, 1, 3),       # temporal pairs only
    (128, (22, 21, 21), 8, 16, 1, 1, 1, 40, 4, 0, 20),   # eight waves
    (128, (22, 21, 21), 5, 17, 1, 16, 1, 3, 3, 2, 1),    # ragged frames, causal blocks of two
])
def test_the_same_bits_as_behind_the_pre_pass(D, pairs, gh, gw, B, H, group, C, Fc, bf, resident):
    import torch
    import paper_2603_17051_amd as A
    w = wl.Workload("rotating", 71, B * group, H, D, gh, gw, C, 0, Fc, resident, pairs)
    q, k, v, do = (dev_bf16(x) for x in wl.chunk_inputs(w, with_dout=True))
    odd = torch.empty(k.numel() + 4, dtype=torch.bfloat16, device="cuda:0")[4:].view(k.shape)  # 8 bytes off
    odd.copy_(k)
    results, staged = [], []
    rotates = Fc * pairs[0] + gh * pairs[1] + gw * pairs[2] <= (896 if D == 128 else 384)  # (cos, sin) the launch has room for
    for keys in (k, odd):
        cache = A.astro_kvcache_create(B, H, D, gh, gw, C, 0, Fc, pairs, w.rope_base, block_frames=bf, reuse_staged=True)
        for b in range(B):
            A.astro_kvcache_reset(cache, b, 5 + 1000 * b)
        frames = [torch.randn((B, gh * gw, H, D), generator=torch.Generator("cuda:0").manual_seed(9), device="cuda:0").bfloat16()] * 2
        for _ in range(resident):
            A.astro_kvcache_append(cache, *frames, 1)
        ws = torch.full((max(A.astro_group_attn_workspace_bytes(cache, Fc, group)),), 255, dtype=torch.uint8, device="cuda:0")
        A.astro_profile_begin()
        out, lse = A.astro_group_attn_fwd(cache, q, keys, v, Fc, group, workspace=ws)
        grads = A.astro_group_attn_bwd(cache, q, keys, v, out, lse, do, Fc, group, workspace=ws)
        launched = A.astro_profile_end()
        if rotates and keys is k:  # one launch, which leaves its operands to the backward
            assert "attn_fwd_few_rotating_bf16" in launched and not {"attn_fwd_few_bf16", "chunk_rope_stage"} & set(launched), launched
        else:
            assert "attn_fwd_few_bf16" in launched and launched["chunk_rope_stage"][0] == 1 and "attn_fwd_few_rotating_bf16" not in launched, launched
        results.append((out, lse) + tuple(grads))
        # rotated queries, rotated keys, and the frames' (cos, sin): each at the next multiple of 256 bytes
        size = (q.numel() * 2 + 255) // 256 * 256
        table = B * group * Fc * max(pairs[0], 1) * 8
        staged.append(torch.cat([ws[:q.numel() * 2], ws[size:size + q.numel() * 2], ws[2 * size:2 * size + (table if pairs[0] else 0)]]))
        torch.cuda.synchronize()
        cache.close()
    for a, b in zip(*results):
        assert torch.equal(a, b)
    assert torch.equal(*staged)

"""Attention over streams of different lengths: the plain order of the workgroups, key ranges that some streams
leave empty, dQ helpers over items of different walks and of several items, ring rows past a short stream's
end.  One head's data repeated over the heads, dO times a power of two of its own for each: every pair is
compared, with the oracle or bit for bit with the pair that was."""
import numpy as np
import pytest

import workloads as wl
from helpers import Lockstep, assert_bf16_close, host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,gh,gw,C,Fc,bf,lens,group,dq_split", [
    (128, 5, 20, 26, 6, 4, 0, [0, 6, 1], 1, True),      # 17 query tiles; the first stream leaves ranges empty; a helper each
    (64, 7, 20, 26, 6, 4, 1, [6, 0, 2, 0], 1, False),
    (128, 9, 20, 26, 6, 4, 0, [6, 1], 2, True),         # two candidates a stream, a helper each, plain order
    (128, 8, 20, 26, 6, 4, 0, [6, 1], 1, True),         # two helpers each
    (128, 3, 10, 13, 8, 3, 1, [0, 8, 3], 1, None),      # few rows
    (64, 16, 16, 20, 9, 2, 0, [9, 1, 0, 0, 4, 2], 1, False),
    (128, 18, 20, 26, 6, 4, 0, [3], 1, True),           # a helper per two items
    (64, 35, 20, 26, 6, 4, 0, [6], 1, True),            # per four
])
def test_streams_of_different_lengths(D, H, gh, gw, C, Fc, bf, lens, group, dq_split):
    import torch
    B = len(lens)
    w = wl.Workload("uneven", 57, B, 1, D, gh, gw, C, 0, Fc, 0, wl.default_rope_pairs(D))
    ls = Lockstep(w, max_chunk=Fc, start_frames=[0] * B, block_frames=bf)   # one head: the oracle
    A = ls.A
    wide = A.astro_kvcache_create(B, H, D, gh, gw, C, 0, Fc, w.rope_pairs, w.rope_base, block_frames=bf)
    rep = lambda x: x.expand(-1, -1, H, -1).contiguous()
    pool_k, pool_v = wl.history_frame_pool(w, 3)
    # a stream of n frames is emptied n steps before the end, so that it holds the last n
    for step in range(max(lens)):
        for b in range(B):
            if lens[b] == max(lens) - step and step > 0:
                for c in (ls.cache, wide):
                    A.astro_kvcache_reset(c, b, 0)
                ls.oracle.reset(b, 0)
        k, v = (np.stack([x[step % 3]] * B) for x in (pool_k, pool_v))
        ls.append(k, v, 1)
        A.astro_kvcache_append(wide, rep(ls.dev(k)), rep(ls.dev(v)), 1)
    for b in range(B):
        if lens[b] == 0:
            for c in (ls.cache, wide):
                A.astro_kvcache_reset(c, b, 0)
            ls.oracle.reset(b, 0)
    assert A.astro_kvcache_tables(wide)[2] == lens
    q, k, v, do = wl.group_inputs(w, group, with_dout=True) if group > 1 else wl.chunk_inputs(w, with_dout=True)
    dev = [rep(ls.dev(x)) for x in (q, k, v, do)]
    nan = lambda dtype, shape: torch.full(shape, float("nan"), dtype=dtype, device="cuda:0")
    out, lse = nan(torch.bfloat16, dev[0].shape), nan(torch.float32, (B * group, H, w.n_q))
    grads = [nan(torch.float32, dev[0].shape) for _ in range(3)]
    factor = 2.0 ** torch.tensor([h % 7 - 3 if h else 0 for h in range(H)], device="cuda:0").view(H, 1)
    dev[3] = dev[3] * factor.bfloat16()
    A.astro_group_attn_fwd(wide, *dev[:3], Fc, group, out, lse)
    A.astro_profile_begin()
    A.astro_group_attn_bwd(wide, *dev[:3], out, lse, dev[3], Fc, group, *grads)
    launched = A.astro_profile_end()
    assert ("attn_bwd_few_bf16" in launched) == (dq_split is None) and ("attn_bwd_dq_merge" in launched) == bool(dq_split), launched
    f64 = [ls.wide(x) for x in (q, k, v, do)]
    ro, rl = ls.oracle.group_attn_fwd(*f64[:3], Fc, group) if group > 1 else ls.oracle.attn_fwd(*f64[:3], Fc)
    rg = ls.oracle.group_attn_bwd(*f64, Fc, group) if group > 1 else ls.oracle.attn_bwd(*f64, Fc)
    for b in range(B * group):
        for got, ref, what in [(out[b, :, 0], ro[b, :, 0], "out"), (lse[b, 0], rl[b, 0], "lse")] + \
                [(g[b, :, 0], r[b, :, 0], n) for g, r, n in zip(grads, rg, ("dq", "dk", "dv"))]:
            assert_bf16_close(host_f64(got), ref, f"candidate {b} {what}")
    # the same inputs on every head: the same bits, the gradients times the head's power of two
    same = lambda x, f=1.0: all(torch.equal(x[:, :, h], x[:, :, 0] * f[h]) for h in range(1, H))
    assert same(out, torch.ones(H, 1, device="cuda:0").bfloat16()) and all(torch.equal(lse[:, h], lse[:, 0]) for h in range(H))
    assert all(same(g, factor) for g in grads)
    if group == 1:
        full = A.astro_chunk_attn_bwd_full(wide, *dev[:3], out, lse, dev[3], Fc)
        extra = ls.oracle.attn_bwd(*f64, Fc, history_grads=True)[3]
        T = w.tokens_per_frame
        for b in range(B):
            if lens[b]:
                assert_bf16_close(host_f64(full[4][b, :lens[b] * T, 0]), extra[(b, 0)]["dv_hist"], f"stream {b} dv_cache")
            assert (full[3][b, lens[b] * T:] == 0).all() and (full[4][b, lens[b] * T:] == 0).all()
        assert same(full[3], factor) and same(full[4], factor)
    wide.close()
    ls.close()

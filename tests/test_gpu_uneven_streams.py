"""Attention over streams of different lengths: the plain order of the workgroups, key ranges that some streams
leave empty, helpers over items of different walks, ring rows past a short stream's end; one chunk repeated over
heads, so that every pair is compared (with the oracle or bit for bit with the pair that was)."""
import numpy as np
import pytest

import workloads as wl
from helpers import Lockstep, assert_bf16_close, host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,gh,gw,C,Fc,bf,lens,group", [
    (128, 5, 20, 26, 6, 4, 0, [0, 6, 1], 1),      # 17 query tiles; the first stream leaves ranges empty
    (64, 7, 20, 26, 6, 4, 1, [6, 0, 2, 0], 1),
    (128, 9, 20, 26, 6, 4, 0, [6, 1], 2),         # two candidates a stream
    (128, 3, 10, 13, 8, 3, 1, [0, 8, 3], 1),      # few rows
    (64, 16, 16, 20, 9, 2, 0, [9, 1, 0, 0, 4, 2], 1),
])
def test_streams_of_different_lengths(D, H, gh, gw, C, Fc, bf, lens, group):
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
        k, v = (np.ascontiguousarray(np.broadcast_to(x[step % 3], (B, *x.shape[1:]))) for x in (pool_k, pool_v))
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
    A.astro_group_attn_fwd(wide, *dev[:3], Fc, group, out, lse)
    A.astro_group_attn_bwd(wide, *dev[:3], out, lse, dev[3], Fc, group, *grads)
    f64 = [ls.wide(x) for x in (q, k, v, do)]
    ro, rl = ls.oracle.group_attn_fwd(*f64[:3], Fc, group) if group > 1 else ls.oracle.attn_fwd(*f64[:3], Fc)
    rg = ls.oracle.group_attn_bwd(*f64, Fc, group) if group > 1 else ls.oracle.attn_bwd(*f64, Fc)
    for b in range(B * group):
        for got, ref, what in [(out[b, :, 0], ro[b, :, 0], "out"), (lse[b, 0], rl[b, 0], "lse")] + \
                [(g[b, :, 0], r[b, :, 0], n) for g, r, n in zip(grads, rg, ("dq", "dk", "dv"))]:
            assert_bf16_close(host_f64(got), ref, f"candidate {b} {what}")
    # the same inputs on every head: the same bits
    for x in [out, *grads]:
        assert all(torch.equal(x[:, :, h], x[:, :, 0]) for h in range(H))
    assert all(torch.equal(lse[:, h], lse[:, 0]) for h in range(H))
    if group == 1:
        full = A.astro_chunk_attn_bwd_full(wide, *dev[:3], out, lse, dev[3], Fc)
        extra = ls.oracle.attn_bwd(*f64, Fc, history_grads=True)[3]
        T = w.tokens_per_frame
        for b in range(B):
            if lens[b]:
                assert_bf16_close(host_f64(full[4][b, :lens[b] * T, 0]), extra[(b, 0)]["dv_hist"], f"stream {b} dv_cache")
            assert (full[3][b, lens[b] * T:] == 0).all() and (full[4][b, lens[b] * T:] == 0).all()
            assert all(torch.equal(full[i][b, :, h], full[i][b, :, 0]) for i in (3, 4) for h in range(H))
    wide.close()
    ls.close()

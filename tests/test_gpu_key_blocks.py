"""The backward's dK and dV over key blocks: at D = 64 with roles, with one wave and with two waves that hold both gradients of a block of
keys, and where ring and chunk go out in one launch (non-detached, not under causal blocks nor by the kernels for few rows), at the
edges of key blocks, query tiles, causal blocks and of the ring, against the fp64 oracle (the gates hold for each
gradient over all its heads); the chunk's are those of the detached backward, whose launch has the chunk only, bit for bit."""
import numpy as np
import pytest

import workloads as wl
from helpers import Lockstep, assert_bf16_close, host_f64
from oracle.rolling_attention import rope_angles, rope_rotate, visible_history
from test_gpu_full_bwd import _slot
from test_gpu_parity import _fill_history

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,gh,gw,C,S,Fc,bf,streamed,only,joint", [
    # one wave a block, chunk of 260 workgroups and more
    (4, 65, 3, 11, 2, 0, 1, 0, 3, None, True),    # one block of 66 ring and 33 chunk rows
    (4, 65, 8, 8, 2, 1, 1, 0, 4, None, True),     # whole tiles, 128 + 64 rows: the chunk begins at a block
    (4, 65, 7, 9, 3, 1, 1, 0, 2, None, True),     # a row short of a tile, one slot empty: two chunk rows in the ring's block
    (2, 65, 10, 13, 3, 0, 1, 0, 3, None, True),   # three query tiles, the last of two rows
    (5, 52, 1, 43, 3, 0, 3, 1, 0, None, False),    # 129 chunk rows in causal blocks of 43, nothing resident
    (5, 52, 1, 43, 3, 0, 3, 1, 3, None, False),    # ... over as many resident: two launches
    # two waves a block, 33 query tiles
    (1, 1, 18, 38, 3, 0, 3, 0, 3, None, True),    # 2052 + 2052 rows: the last tile has four, the chunk begins inside a block
    (1, 1, 18, 38, 3, 0, 3, 1, 3, None, False),    # causal blocks: two launches
    (1, 1, 22, 32, 3, 0, 3, 0, 2, None, True),    # whole tiles of 64, the chunk begins at a block
    (3, 2, 18, 38, 3, 0, 3, 0, 2, 2, True),       # streams of different lengths: the last one is empty
    (1, 1, 12, 35, 4, 1, 2, 0, 6, None, False),    # 14 tiles, the chunk by the kernel for few rows: the ring by itself
    # roles
    (2, 65, 6, 7, 3, 0, 1, 0, 4, None, False),     # ring of 130 workgroups
    (1, 129, 1, 1, 100, 0, 1, 0, 70, None, False), # ... of 129, frames of one token: the table of frames behind the walk
    (1, 65, 10, 13, 20, 1, 1, 0, 23, None, False), # chunk of 130; ring of 1365 by one wave
    (1, 65, 5, 13, 40, 0, 2, 1, 40, None, False),  # the same under causal blocks
    (2, 65, 1, 43, 3, 1, 2, 1, 5, None, False),    # few chunk rows, ring of 260 workgroups by one wave
])
def test_both_gradients_of_a_block_at_64(B, H, gh, gw, C, S, Fc, bf, streamed, only, joint):
    check(64, (12, 10, 10), B, H, gh, gw, C, S, Fc, bf, streamed, only, joint)


@pytest.mark.parametrize("B,H,gh,gw,C,S,Fc,bf,streamed,only,joint", [
    (2, 73, 3, 11, 2, 0, 1, 0, 3, 2, True),    # one block of 66 ring and 33 chunk rows
    (2, 73, 1, 43, 3, 1, 2, 1, 5, 2, False),    # causal blocks: two launches
    (2, 73, 8, 8, 2, 0, 1, 0, 2, 2, True),     # the chunk begins at a block
    (3, 49, 6, 7, 4, 1, 2, 0, 6, 2, True),     # streams of different lengths: the last one is empty
    (3, 49, 6, 7, 4, 1, 2, 1, 6, 2, False),    # ... under causal blocks: two launches
    (1, 146, 7, 9, 3, 1, 1, 0, 0, 1, False),    # nothing resident: a launch of its own
])
def test_ring_and_chunk_in_one_launch(B, H, gh, gw, C, S, Fc, bf, streamed, only, joint):
    check(128, (22, 21, 21), B, H, gh, gw, C, S, Fc, bf, streamed, only, joint)


def check(D, pairs, B, H, gh, gw, C, S, Fc, bf, streamed, only, joint):
    """`only`: streams with history, None = all; `joint`: whether the ring's and the chunk's are one launch"""
    T = gh * gw
    w = wl.Workload("key_blocks", 57, B, H, D, gh, gw, C, S, Fc, streamed, pairs)
    ls = Lockstep(w, max_chunk=Fc, start_frames=[3 + 100 * b for b in range(B)], block_frames=bf)
    _fill_history(ls, w, *wl.history_frame_pool(w, 7), streamed)
    n = [streamed if only is None or b < only else 0 for b in range(B)]
    for b in range(B):
        if n[b] != streamed:
            ls.A.astro_kvcache_reset(ls.cache, b, 3 + 100 * b)
            ls.oracle.reset(b, 3 + 100 * b)
    q, k, v, do = wl.chunk_inputs(w, with_dout=True)
    out, lse = ls.fwd(q, k, v, Fc)
    ls.A.astro_profile_begin()
    _, dk, dv, dkc, dvc = ls.A.astro_chunk_attn_bwd_full(ls.cache, *[ls.dev(x) for x in (q, k, v)], out, lse, ls.dev(do), Fc)
    launched = ls.A.astro_profile_end()
    assert ("attn_bwd_dkv_joint_bf16" in launched) == joint and ("attn_bwd_dkv_hist_bf16" in launched) == (streamed > 0 and not joint), launched
    detached = ls.A.astro_chunk_attn_bwd(ls.cache, *[ls.dev(x) for x in (q, k, v)], out, lse, ls.dev(do), Fc)
    assert dk.equal(detached[1]) and dv.equal(detached[2])
    _, rk, rv, extra = ls.oracle.attn_bwd(*[ls.wide(x) for x in (q, k, v, do)], Fc, history_grads=True)
    assert_bf16_close(host_f64(dk), rk, "dk")
    assert_bf16_close(host_f64(dv), rv, "dv")
    ref_k, ref_v = np.zeros((B, C * T, H, D)), np.zeros((B, C * T, H, D))
    for b in range(B):
        for i, f in enumerate(visible_history(n[b], S, C - S)):
            rows = slice(_slot(f, C, S) * T, (_slot(f, C, S) + 1) * T)
            phi = rope_angles(ls.oracle.start[b] + f, gh, gw, w.rope_pairs, w.rope_base)
            for h in range(H):
                ref_k[b, rows, h] = rope_rotate(extra[(b, h)]["dk_hist_rot"][i * T:(i + 1) * T, None, :], -phi)[:, 0]
                ref_v[b, rows, h] = extra[(b, h)]["dv_hist"][i * T:(i + 1) * T]
    if streamed:
        assert_bf16_close(host_f64(dkc), ref_k, "dk_cache")
        assert_bf16_close(host_f64(dvc), ref_v, "dv_cache")
    else:
        assert (dkc == 0).all() and (dvc == 0).all()
    ls.close()


@pytest.mark.parametrize("D,pairs,B,H", [(64, (12, 10, 10), 2, 65), (128, (22, 21, 21), 1, 73)])
def test_a_gradient_that_is_not_finite_reaches_the_same_chunk_keys_as_detached(D, pairs, B, H):
    """Causal frames of 65 tokens behind one resident: no key of the second block of 128 chunk rows is seen by the first tile of
    queries.  Where a query of that tile has infinite output gradients, theirs stay what they are without it."""
    Fc, T, C = 3, 65, 3
    w = wl.Workload("not_finite", 58, B, H, D, 5, 13, C, 0, Fc, 1, pairs)
    ls = Lockstep(w, max_chunk=Fc, start_frames=[3 + b for b in range(B)], block_frames=1)
    _fill_history(ls, w, *wl.history_frame_pool(w, 3), 1)
    q, k, v, do = wl.chunk_inputs(w, with_dout=True)
    dev = [ls.dev(x) for x in (q, k, v)]
    out, lse = ls.fwd(q, k, v, Fc)
    dout = ls.dev(do)
    clean = ls.A.astro_chunk_attn_bwd(ls.cache, *dev, out, lse, dout, Fc)
    dout[:, 10] = float("inf")
    detached = ls.A.astro_chunk_attn_bwd(ls.cache, *dev, out, lse, dout, Fc)
    full = ls.A.astro_chunk_attn_bwd_full(ls.cache, *dev, out, lse, dout, Fc)
    for kept, got, want in zip(clean[1:], full[1:3], detached[1:]):
        assert (got.isfinite() == want.isfinite()).all()
        assert got[:, 2 * T:].equal(kept[:, 2 * T:]) and not got[:, :T].isfinite().any()
    ls.close()

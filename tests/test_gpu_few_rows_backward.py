"""The backward's kernel for few rows at the sizes where its shared operands, row terms and rotary look-ups can go
wrong: one row, rows around a trip of the row terms, the most rows it takes, both numbers of waves, no rotary pairs;
fp64 oracle, outputs pre-filled with NaN.  And, on the CPU, the division by reciprocal behind the look-ups."""
import numpy as np
import pytest

import workloads as wl
from helpers import Lockstep, assert_bf16_close, host_f64
from test_gpu_parity import _fill_history

P64, P128, NONE = (12, 10, 10), (22, 21, 21), (0, 0, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("D,pairs,gh,gw,B,H,C,Fc,bf,resident", [
    (64, P64, 5, 13, 1, 2, 3, 2, 0, 3),       # 130 rows: one past a trip of the row terms (128 rows, four waves)
    (128, P128, 5, 13, 1, 2, 3, 1, 0, 3),     # 65 rows: the same with 64
    (128, NONE, 5, 13, 1, 2, 3, 2, 1, 3),     # nothing to turn back
    (64, P64, 32, 64, 1, 1, 2, 1, 0, 1),      # the most rows: eight waves
    (128, P128, 31, 66, 1, 1, 2, 1, 0, 1),    # 2046 of them, ragged
    (64, NONE, 16, 24, 2, 1, 4, 2, 1, 4),     # eight waves, causal, streams two
    (128, P128, 11, 23, 1, 3, 5, 3, 0, 5),    # eight waves, ragged frames, row terms in a launch before
    (64, P64, 19, 27, 2, 3, 3, 2, 1, 1),      # the same at D = 64, causal, streams two
    (128, P128, 16, 24, 1, 2, 4, 1, 0, 3),    # 384 rows over 1152 of the ring: within the launch
])
def test_backward_with_few_rows(D, pairs, gh, gw, B, H, C, Fc, bf, resident):
    import torch
    w = wl.Workload("few_rows_bwd", 71, B, H, D, gh, gw, C, 0, Fc, resident, pairs)
    ls = Lockstep(w, max_chunk=Fc, start_frames=[5 + 9 * b for b in range(B)], block_frames=bf)
    _fill_history(ls, w, *wl.history_frame_pool(w, 3), resident)
    q, k, v, do = wl.chunk_inputs(w, with_dout=True)
    dev = [ls.dev(x) for x in (q, k, v, do)]
    grads = [torch.full(dev[0].shape, float("nan"), dtype=torch.float32, device="cuda:0") for _ in range(3)]
    ls.A.astro_profile_begin()
    out, lse = ls.A.astro_chunk_attn_fwd(ls.cache, *dev[:3], Fc)
    ls.A.astro_chunk_attn_bwd(ls.cache, *dev[:3], out, lse, dev[3], Fc, *grads)
    launched = ls.A.astro_profile_end()
    ring = resident * gh * gw
    assert "attn_bwd_few_bf16" in launched
    assert ("attn_bwd_few_row_terms" in launched) == (w.n_q >= 384 and ring < 3 * w.n_q if D == 128 else w.n_q >= 512 and ring < 2 * w.n_q)
    wide = [ls.wide(x) for x in (q, k, v, do)]
    for b, h in {(0, 0), (B - 1, H - 1)}:
        ref = ls.oracle.attn_bwd(*wide, Fc, streams=[b], heads=[h])
        for g, r, n in zip(grads, ref, ("dq", "dk", "dv")):
            assert_bf16_close(host_f64(g[b, :, h]), r[b, :, h], f"pair {b, h} {n}")
    assert all(bool(torch.isfinite(x).all()) for x in grads)
    ls.close()


def test_quotients_by_reciprocal_are_exact():
    """A token's frame and row: (n + 1/2) times a reciprocal that is off by up to two units in the last place."""
    n = np.arange(2048, dtype=np.int64)
    half = n.astype(np.float32) + np.float32(0.5)
    for d in range(1, 2049):
        r = np.float32(1) / np.float32(d)
        for x in (np.nextafter(np.nextafter(r, np.float32(0)), np.float32(0)), r, np.nextafter(np.nextafter(r, np.float32(2)), np.float32(2))):
            assert np.array_equal((half * x).astype(np.int64), n // d), d

"""Ring-row gradients of the non-detached backward where many frames share a workgroup's 128 keys: the
table of temporal factors that fits beside the tiles, and the one that does not (one-token frames with
all pairs on the frame axis); wrapped rings with sinks, against the fp64 oracle."""
import pytest

import workloads as wl
from helpers import Lockstep, assert_bf16_close, host_f64
from test_gpu_full_bwd import _check_ring_grads
from test_gpu_parity import _fill_history

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,pairs,gh,gw,C,S,Fc,streamed", [
    (128, (64, 0, 0), 1, 1, 150, 3, 40, 170),   # 128 frames x 64 pairs: 64 KB, twice a tile slot
    (64, (32, 0, 0), 1, 1, 150, 0, 40, 150),    # 128 x 32: 32 KB, twice a tile slot at D 64
    (128, (22, 21, 21), 2, 3, 40, 2, 8, 60),    # six-token frames: 22 in a workgroup, boundaries inside it
    (64, (12, 10, 10), 1, 3, 50, 1, 30, 50),
])
def test_ring_gradients_with_many_frames_per_workgroup(D, pairs, gh, gw, C, S, Fc, streamed):
    w = wl.Workload("ring_grads", 52, 2, 1, D, gh, gw, C, S, Fc, streamed, pairs)
    ls = Lockstep(w, max_chunk=Fc, start_frames=[5, 1000])
    _fill_history(ls, w, *wl.history_frame_pool(w, 7), streamed)
    q, k, v, do = wl.chunk_inputs(w, with_dout=True)
    out, lse = ls.fwd(q, k, v, Fc)
    _, dk, _, dkc, dvc = ls.A.astro_chunk_attn_bwd_full(ls.cache, *[ls.dev(x) for x in (q, k, v)], out, lse, ls.dev(do), Fc)
    _, rk, _, extra = ls.oracle.attn_bwd(*[ls.wide(x) for x in (q, k, v, do)], Fc, history_grads=True)
    assert_bf16_close(host_f64(dk), rk, "dk")
    _check_ring_grads(ls, dkc, dvc, extra, [(0, 0), (1, 0)], [], "ring")
    ls.close()

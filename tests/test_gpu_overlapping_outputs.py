"""Gradients written over memory that the call still reads on another route: the launches that take both sides
at once or pass partial sums through dK and dV leave such calls to the two plain launches, whose first
reads it all.  Each layout at a size of either route, against the fp64 oracle."""
import pytest

import workloads as wl
from helpers import Lockstep, assert_bf16_close, host_f64
from test_gpu_parity import _fill_history

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H,gh,gw,resident,apart", [
    (128, 2, 7, 9, 3, "attn_bwd_few_bf16"),    # few rows
    (128, 1, 20, 26, 2, "attn_bwd_dq_merge"),  # dQ walk in three
    (64, 6, 20, 26, 3, "attn_bwd_dq_merge"),   # in two
])
@pytest.mark.parametrize("layout", ["apart", "one buffer for dk and dv", "dk over out, dv over lse", "dk over dq"])
def test_backward_outputs_over_memory_the_query_side_reads(D, H, gh, gw, resident, apart, layout):
    import torch
    Fc = 4
    w = wl.Workload("overlap", 54, 1, H, D, gh, gw, 4, 0, Fc, resident, wl.default_rope_pairs(D))
    ls = Lockstep(w, max_chunk=Fc, start_frames=[9])
    _fill_history(ls, w, *wl.history_frame_pool(w, 3), resident)
    q, k, v, do = wl.chunk_inputs(w, with_dout=True)
    dev = [ls.dev(x) for x in (q, k, v, do)]
    out, lse = ls.A.astro_chunk_attn_fwd(ls.cache, *dev[:3], Fc)
    dq, dk, dv = [torch.full(dev[0].shape, float("nan"), device="cuda:0") for _ in range(3)]
    wanted = "qkv"
    if layout == "one buffer for dk and dv":
        dv, wanted = dk, "q"
    elif layout == "dk over dq":
        dk, wanted = dq, "kv"
    elif layout == "dk over out, dv over lse":
        shared = dk.view(-1)[dk.numel() // 2:].view(torch.bfloat16).view(out.shape)  # the second half of dk's bytes
        shared.copy_(out)
        terms = dv.view(-1)[:lse.numel()].view(lse.shape)
        terms.copy_(lse)
        out, lse = shared, terms
    ls.A.astro_profile_begin()
    ls.A.astro_chunk_attn_bwd(ls.cache, *dev[:3], out, lse, dev[3], Fc, dq, dk, dv)
    launched = ls.A.astro_profile_end()
    assert (apart in launched) == (layout == "apart"), launched
    ref = ls.oracle.attn_bwd(*[ls.wide(x) for x in (q, k, v, do)], Fc, heads=[H - 1])
    for got, r, what in zip((dq, dk, dv), ref, "qkv"):
        if what in wanted:
            assert_bf16_close(host_f64(got[0, :, H - 1]), r[0, :, H - 1], f"{layout}: d{what}")
    ls.close()

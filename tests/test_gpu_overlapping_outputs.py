"""Outputs over memory that the call still reads on another route: such calls take the route that reads it all
first (backward: the two plain launches instead of one for both sides or partial sums in dK and dV, and
ring and chunk in a launch each; forward: key ranges merged at the end).  Each layout at a size of either route, against the fp64 oracle."""
import numpy as np
import pytest

import workloads as wl
from helpers import Lockstep, assert_bf16_close, host_f64
from oracle import rope_angles, rope_rotate
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


@pytest.mark.parametrize("H,gh,gw,resident,apart", [
    (2, 7, 9, 3, "attn_fwd_few_rotating_bf16"),
    (12, 30, 36, 2, "attn_fwd_merge"),  # 408 workgroups
])
def test_forward_in_place_of_the_chunk_values(H, gh, gw, resident, apart):
    D, Fc = 128, 4
    w = wl.Workload("overlap_fwd", 55, 1, H, D, gh, gw, 4, 0, Fc, resident, wl.default_rope_pairs(D))
    ls = Lockstep(w, max_chunk=Fc, start_frames=[9])
    _fill_history(ls, w, *wl.history_frame_pool(w, 3), resident)
    q, k, v = wl.chunk_inputs(w)
    ref, ref_lse = ls.oracle.attn_fwd(*[ls.wide(x) for x in (q, k, v)], Fc, heads=[H - 1])
    for in_place in (False, True):
        dev = [ls.dev(x) for x in (q, k, v)]
        ls.A.astro_profile_begin()
        out, lse = ls.A.astro_chunk_attn_fwd(ls.cache, *dev, Fc, out=dev[2] if in_place else None)
        launched = ls.A.astro_profile_end()
        assert ("attn_fwd_merge" if in_place else apart) in launched, launched
        assert_bf16_close(host_f64(out[0, :, H - 1]), ref[0, :, H - 1], f"in place {in_place}: out")
        assert_bf16_close(host_f64(lse[0, H - 1]), ref_lse[0, H - 1], f"in place {in_place}: lse")
    ls.close()


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("layout", ["apart", "out over q", "out over k", "lse in q", "lse in k"])
def test_few_rows_forward_with_outputs_over_its_queries_and_keys(D, layout):
    """A launch that rotates for itself reads both to its end, by every workgroup of a pair: such calls go behind
    the pre-pass, which has read them before the first output is written."""
    import torch
    Fc = 4
    w = wl.Workload("overlap_chunk", 57, 1, 2, D, 7, 9, 4, 0, Fc, 3, wl.default_rope_pairs(D))
    ls = Lockstep(w, max_chunk=Fc, start_frames=[9])
    _fill_history(ls, w, *wl.history_frame_pool(w, 3), 3)
    q, k, v = wl.chunk_inputs(w)
    dq, dk, dv = (ls.dev(x) for x in (q, k, v))
    into = dq if layout.endswith("q") else dk
    out = into if layout.startswith("out") else torch.empty_like(dq)
    lse = torch.empty((1, 2, w.n_q), device="cuda:0")
    if layout.startswith("lse"):  # the bytes of rows in the middle
        lse = into.view(-1)[into.numel() // 2:into.numel() // 2 + 2 * lse.numel()].view(torch.float32).view(lse.shape)
    ls.A.astro_profile_begin()
    ls.A.astro_chunk_attn_fwd(ls.cache, dq, dk, dv, Fc, out, lse)
    launched = ls.A.astro_profile_end()
    assert set(launched) == ({"attn_fwd_few_rotating_bf16"} if layout == "apart" else {"chunk_rope_stage", "attn_fwd_few_bf16"}), launched
    ref, ref_lse = ls.oracle.attn_fwd(*[ls.wide(x) for x in (q, k, v)], Fc)
    assert_bf16_close(host_f64(out), ref, f"{layout}: out")
    assert_bf16_close(host_f64(lse), ref_lse, f"{layout}: lse")
    ls.close()


@pytest.mark.parametrize("D,window_relative", [(128, False), (64, True)])
@pytest.mark.parametrize("layout", ["one buffer for dk_cache and dv_cache", "dk_cache over dout", "dk_cache over dout and dv_cache"])
def test_ring_gradients_over_each_other_and_over_dout(D, window_relative, layout):
    import torch
    Fc, C = 2, 5
    w = wl.Workload("overlap_ring", 56, 2, 2, D, 7, 9, C, 1, Fc, 7, wl.default_rope_pairs(D))
    ls = Lockstep(w, max_chunk=Fc, start_frames=[9, 2], window_relative=window_relative)
    _fill_history(ls, w, *wl.history_frame_pool(w, 3), 7)
    q, k, v, do = wl.chunk_inputs(w, with_dout=True)
    dev = [ls.dev(x) for x in (q, k, v, do)]
    out, lse = ls.A.astro_chunk_attn_fwd(ls.cache, *dev[:3], Fc)
    want = ls.A.astro_chunk_attn_bwd_full(ls.cache, *dev[:3], out, lse, dev[3], Fc)
    dkc = torch.full_like(want[3], float("nan"))
    dvc = torch.full_like(want[4], float("nan")) if layout == "dk_cache over dout" else dkc
    dout = dev[3]
    if "dout" in layout:
        dout = dkc.view(-1).view(torch.bfloat16)[-dout.numel():].view(dout.shape)
        dout.copy_(dev[3])
    got = ls.A.astro_chunk_attn_bwd_full(ls.cache, *dev[:3], out, lse, dout, Fc, dk_cache=dkc, dv_cache=dvc)
    assert all(torch.equal(a, b) for a, b in zip(got[:4], want[:4]))  # the same kernels in the same order of sums
    if dvc is not dkc:
        assert torch.equal(dvc, want[4])
    ls.close()


@pytest.mark.parametrize("D,B,H,gh,gw,C,Fc,resident", [
    (128, 2, 73, 3, 11, 2, 1, 2),
    (64, 4, 65, 3, 11, 2, 1, 2),   # one wave a block of keys
    (64, 1, 2, 18, 38, 3, 3, 2),   # two
])
@pytest.mark.parametrize("layout", ["apart", "one buffer for dk_cache and dv_cache", "dk_cache over dout", "dk_cache over dout and dv_cache",
                                    "dv_cache over dk_chunk"])
def test_ring_gradients_of_calls_that_are_one_launch_otherwise(D, B, H, gh, gw, C, Fc, resident, layout):
    """Sizes at which ring and chunk go out together where nothing overlaps."""
    import torch
    T, pairs = gh * gw, wl.default_rope_pairs(D)
    w = wl.Workload("overlap_joint", 59, B, H, D, gh, gw, C, 0, Fc, resident, pairs)
    ls = Lockstep(w, max_chunk=Fc, start_frames=[9 + b for b in range(B)])
    _fill_history(ls, w, *wl.history_frame_pool(w, 3), resident)
    q, k, v, do = wl.chunk_inputs(w, with_dout=True)
    dev = [ls.dev(x) for x in (q, k, v, do)]
    out, lse = ls.A.astro_chunk_attn_fwd(ls.cache, *dev[:3], Fc)
    detached = ls.A.astro_chunk_attn_bwd(ls.cache, *dev[:3], out, lse, dev[3], Fc)
    nan = lambda *shape: torch.full(shape, float("nan"), device="cuda:0")
    dq, dk, dv, dkc, dvc = [nan(*dev[0].shape) for _ in range(3)] + [nan(B, C * T, H, D) for _ in range(2)]
    dout, wanted = dev[3], {"dq", "dk", "dv", "dk_cache", "dv_cache"}
    if "dout" in layout:
        dout = dkc.view(-1).view(torch.bfloat16)[-dout.numel():].view(dout.shape)
        dout.copy_(dev[3])
    if layout == "dv_cache over dk_chunk":
        dk, wanted = dvc.view(-1)[-dk.numel():].view(dk.shape), wanted - {"dk"}
    elif "dv_cache" in layout:
        dvc, wanted = dkc, wanted - {"dv_cache"}
    ls.A.astro_profile_begin()
    ls.A.astro_chunk_attn_bwd_full(ls.cache, *dev[:3], out, lse, dout, Fc, dq, dk, dv, dkc, dvc)
    launched = ls.A.astro_profile_end()
    assert ("attn_bwd_dkv_joint_bf16" in launched) == (layout == "apart"), launched
    for name, got, want in zip(("dq", "dk", "dv"), (dq, dk, dv), detached):
        assert name not in wanted or got.equal(want), name
    b, h = B - 1, H - 1
    extra = ls.oracle.attn_bwd(*[ls.wide(x) for x in (q, k, v, do)], Fc, streams=[b], heads=[h], history_grads=True)[3][(b, h)]
    rows = resident * T
    if "dk_cache" in wanted:
        ref = np.concatenate([rope_rotate(extra["dk_hist_rot"][f * T:(f + 1) * T, None, :], -rope_angles(ls.oracle.start[b] + f, gh, gw, pairs, w.rope_base))[:, 0]
                              for f in range(resident)])
        assert_bf16_close(host_f64(dkc[b, :rows, h]), ref, f"{layout}: dk_cache")
    if "dv_cache" in wanted:
        assert_bf16_close(host_f64(dvc[b, :rows, h]), extra["dv_hist"], f"{layout}: dv_cache")
    ls.close()

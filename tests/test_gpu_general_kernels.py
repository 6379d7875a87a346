"""The general forward and dQ kernels at inputs that move or strain the softmax reference, unsplit and split: logits that
rise or fall by tens of natural units between frames, logits of about -128 with ragged key tiles, causal ranges that
a query or a whole workgroup sees nothing of.  Small chunks take the kernels for few rows, so these have one
head's data repeated over enough heads (or enough frames); the launch names are asserted, every head is compared bit
for bit with the one that is judged, by the bf16 rounding model on the same inputs."""
import numpy as np
import pytest

import workloads as wl
from bf16_model import model_fwd_bwd
from helpers import Lockstep, assert_bf16_close, assert_within_model, host_f64

pytestmark = pytest.mark.gpu


class Wide:
    """A one-head cache with its oracle, and a cache of H heads that all hold the same frames."""

    def __init__(self, w, H, Fc, bf=0):
        self.ls, self.H = Lockstep(w, max_chunk=Fc, block_frames=bf), H
        self.A = self.ls.A
        self.cache = self.A.astro_kvcache_create(w.batch, H, w.head_dim, w.grid_h, w.grid_w, w.capacity_frames, w.sink_frames, Fc,
                                                 w.rope_pairs, w.rope_base, block_frames=bf)

    def dev(self, x):
        return self.ls.dev(x).expand(-1, -1, self.H, -1).contiguous()

    def append(self, k, v):
        self.ls.oracle.append(self.ls.wide(k), self.ls.wide(v), 1)
        self.A.astro_kvcache_append(self.cache, self.dev(k), self.dev(v), 1)

    def close(self):
        self.cache.close()
        self.ls.close()


def _names(launched, fwd_split, dq_split):
    assert "attn_fwd_bf16" in launched and ("attn_fwd_merge" in launched) == fwd_split, launched
    assert "attn_bwd_dq_bf16" in launched and ("attn_bwd_dq_merge" in launched) == dq_split, launched


# D, heads, token grid, frames in the ring, frames per level, split; logits move by 40 natural units a level
SHAPES = [
    (128, 640, 4, 8, 5, 1, False),
    (64, 1000, 5, 9, 4, 1, False),
    (128, 120, 8, 8, 104, 13, True),
    (64, 136, 8, 8, 120, 15, True),
    (128, 640, 5, 9, 4, 1, False),     # 45-token frames: ragged tiles
    (64, 170, 5, 13, 120, 15, True),   # 65-token frames
]


@pytest.mark.parametrize("D,H,gh,gw,C,per_level,split", SHAPES)
@pytest.mark.parametrize("kind", ["rising", "falling", "negative"])
def test_reference_of_the_general_kernels(D, H, gh, gw, C, per_level, split, kind):
    import torch
    w = wl.Workload("general_ref", 58, 1, 1, D, gh, gw, C, 0, 1, 0, (0, 0, 0))
    x = Wide(w, H, 1)
    step = 40.0 / np.sqrt(D)
    top = C // per_level

    def inputs(i):
        n = [wl.normal_f32(w.seed, t, (1, w.n_q, 1, D), i) for t in (wl.T_Q, wl.T_K, wl.T_V, wl.T_DO)]
        level = i // per_level
        if kind == "negative":   # every logit about -128
            q, k = 128.0 / np.sqrt(D) / 4.0 + 0.5 * n[0], -4.0 - 0.5 * n[1]
        else:
            q, k = 1.0 + 0.5 * n[0], step * (level if kind == "rising" else top - level) + 0.5 * n[1]
        return [wl.f32_to_bf16_bits(v.astype(np.float32)) for v in (q, k, n[2], n[3])]

    for i in range(C):
        _, k, v, _ = inputs(i)
        x.append(k, v)
    q, k, v, do = inputs(C)
    dev = [x.dev(t) for t in (q, k, v, do)]
    nan = lambda dtype, shape: torch.full(shape, float("nan"), dtype=dtype, device="cuda:0")
    out, lse = nan(torch.bfloat16, dev[0].shape), nan(torch.float32, (1, H, w.n_q))
    grads = [nan(torch.float32, dev[0].shape) for _ in range(3)]
    x.A.astro_profile_begin()
    x.A.astro_chunk_attn_fwd(x.cache, *dev[:3], 1, out, lse)
    x.A.astro_chunk_attn_bwd(x.cache, *dev[:3], out, lse, dev[3], 1, *grads)
    _names(x.A.astro_profile_end(), split, split)
    f64 = [x.ls.wide(t) for t in (q, k, v, do)]
    ro, rl = x.ls.oracle.attn_fwd(*f64[:3], 1)
    ref = [ro[0, :, 0], rl[0, 0]] + [g[0, :, 0] for g in x.ls.oracle.attn_bwd(*f64, 1)]
    model = model_fwd_bwd(x.ls.oracle, *f64, 1, 0, 0)
    got = [out[0, :, 0], lse[0, 0]] + [g[0, :, 0] for g in grads]
    for a, r, m, what in zip(got, ref, model, ("out", "lse", "dq", "dk", "dv")):
        assert_within_model(host_f64(a), r, m, f"{kind} {what}")
    if kind == "negative":
        assert rl.max() < -100.0
    else:
        assert np.abs(rl).max() > 60.0
    for t in [out] + grads:
        assert bool((t == t[:, :, :1]).all())
    assert bool((lse == lse[:, :1]).all())
    x.close()


def test_causal_ranges_of_the_split_forward_that_are_empty_or_unseen():
    """37 frames of 100 tokens, frame by frame, on an empty ring: the first query tile sees 7 key tiles of 116 (an empty
    range among the eight), and ranges hold keys of later frames only for some of a workgroup's queries."""
    import torch
    w = wl.Workload("general_unseen", 59, 1, 1, 128, 10, 10, 40, 0, 37, 0, (22, 21, 21))
    ls = Lockstep(w, max_chunk=37, block_frames=1)
    q, k, v, do = wl.chunk_inputs(w, with_dout=True)
    dev = [ls.dev(t) for t in (q, k, v, do)]
    out = torch.full(dev[0].shape, float("nan"), dtype=torch.bfloat16, device="cuda:0")
    lse = torch.full((1, 1, w.n_q), float("nan"), device="cuda:0")
    ls.A.astro_profile_begin()
    ls.A.astro_chunk_attn_fwd(ls.cache, *dev[:3], 37, out, lse)
    grads = ls.A.astro_chunk_attn_bwd(ls.cache, *dev[:3], out, lse, dev[3], 37)
    _names(ls.A.astro_profile_end(), True, True)
    f64 = [ls.wide(t) for t in (q, k, v, do)]
    ro, rl = ls.oracle.attn_fwd(*f64[:3], 37)
    assert_bf16_close(host_f64(out), ro, "out")
    assert_bf16_close(host_f64(lse), rl, "lse")
    for got, r, what in zip(grads, ls.oracle.attn_bwd(*f64, 37), ("dq", "dk", "dv")):
        assert_bf16_close(host_f64(got), r, what)
    ls.close()


def test_causal_ranges_with_64_wide_heads():
    """The same with 97 frames (the forward with few rows takes shorter walks at D = 64); rows of the first frames,
    around the query tiles of later ones, and at the end."""
    w = wl.Workload("general_unseen64", 60, 1, 1, 64, 10, 10, 100, 0, 97, 0, (12, 10, 10))
    ls = Lockstep(w, max_chunk=97, block_frames=1)
    q, k, v = wl.chunk_inputs(w)
    ls.A.astro_profile_begin()
    out, lse = ls.fwd(q, k, v, 97)
    launched = ls.A.astro_profile_end()
    assert "attn_fwd_bf16" in launched and "attn_fwd_merge" in launched, launched
    rows = np.unique(np.concatenate([np.arange(0, 400), np.arange(1270, 1300), np.arange(4860, 4920), np.arange(9600, 9700)]))
    ro, rl = ls.oracle.attn_fwd(*[ls.wide(t) for t in (q, k, v)], 97, rows=rows)
    assert_bf16_close(host_f64(out[0, rows, 0]), ro[0, rows, 0], "out")
    assert_bf16_close(host_f64(lse[0, 0, rows]), rl[0, 0, rows], "lse")
    ls.close()

"""The work a program has this library do, as timed cases.

Every case goes through the package's public entry points with bf16 caches (the fp32 cache is a
debug path: it keeps a score matrix in memory and is only used to check results).  Kinds:

  forward   one chunk attention over the rolling cache (a denoising step of a rollout); with
            group > 1, the candidates of one group over their shared, frozen cache
  update    forward, then the backward with the cached context detached, on one chunk (the
            re-forward + backward of gradient checkpointing in a clip-window update; the handle
            may reuse what the forward staged)
  full      the same with the non-detached backward: ring rows get gradients as well
  rollout   a new video: reset, then for every chunk attention followed by the append; the ring
            fills, evicts, and with window-relative positions the sinks move
  prefill   rebuild a cache from known frames: reset, then nothing but appends
  loss      the fused clip-level loss and its gradient

Values are N(0,1) rounded to bf16, as in the repository's benchmark.
"""
import math

import torch

import paper_2603_17051_amd as A

DEV = "cuda:0"
ROPE_BASE = 10000.0
A_MAX, BETA, LAMBDA_KL = 1.2, 1.0, 0.1


def _attention(name, kind, batch, heads, head_dim, grid_h, grid_w, capacity, sinks, chunk, streamed, group=1, block=0,
               relative=False, chunks=1):
    """streamed: frames appended before the measured chunk; chunks: chunks of a rollout or prefill."""
    c = dict(kind=kind, batch=batch, heads=heads, head_dim=head_dim, grid_h=grid_h, grid_w=grid_w, capacity=capacity,
             sinks=sinks, chunk=chunk, streamed=streamed, group=group, block=block, relative=relative, chunks=chunks)
    return dict(name=name, **c) if name else c


def _loss(name, clips, elems, dtype):
    c = dict(kind="loss", clips=clips, elems=elems, dtype=dtype)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest configuration: one 64-token frame over a full ring of four (unit-sized models, latency)
        _attention("tiny_forward", "forward", 1, 2, 64, 8, 8, 4, 0, 1, 4),
        _attention("tiny_update", "update", 1, 2, 64, 8, 8, 4, 0, 1, 4),
        # a small model in development: ragged frames of 130 tokens, a sink, a ring that has wrapped
        _attention("small_update_d64", "update", 2, 8, 64, 10, 13, 6, 1, 2, 9),
        # a mid-sized model with frame-causal chunks: the production grid with 64-wide heads
        _attention("causal_update_d64", "update", 1, 16, 64, 30, 52, 12, 1, 3, 14, block=1),
        # the production layer, one stream: what serving a single video runs per layer and step
        _attention("production_forward", "forward", 1, 12, 128, 30, 52, 18, 0, 3, 18),
        # ... and what a training rank with one clip per step runs per layer
        _attention("production_update", "update", 1, 12, 128, 30, 52, 18, 0, 3, 18),
        # the benchmark's step: four clips
        _attention("batch4_update", "update", 4, 12, 128, 30, 52, 18, 0, 3, 18),
        # group sampling: eight candidate chunks over one shared cache
        _attention("group8_forward", "forward", 1, 12, 128, 30, 52, 18, 0, 3, 18, group=8),
        # training without the detach
        _attention("production_full", "full", 1, 12, 128, 30, 52, 18, 0, 3, 18),
        # long streaming: ring of 12 with one sink and window-relative positions, 6 chunks from an empty cache
        _attention("stream_rollout", "rollout", 1, 12, 128, 30, 52, 12, 1, 3, 0, relative=True, chunks=6),
        # rebuilding eight caches of 18 frames before a clip window is trained
        _attention("batch8_prefill", "prefill", 8, 12, 128, 30, 52, 18, 0, 3, 0, chunks=6),
        # the loss of one group of 24 clips (three latent frames of 16 x 60 x 104 each)
        _loss("group24_loss", 24, 3 * 16 * 60 * 104, "bf16"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    most = max(work(c)["flops"] for c in listed())
    most_bytes = max(work(c)["bytes"] for c in listed())
    while True:
        kind = rng.choice(["forward", "forward", "update", "update", "update", "full", "rollout", "prefill", "loss"])
        if kind == "loss":
            c = _loss(None, _log_int(rng, 1, 192), 8 * _log_int(rng, 64, 3 * 16 * 60 * 104 // 8),
                      rng.choice(["bf16", "bf16", "f32"]))
        else:
            capacity = rng.randint(2, 18)
            sinks = rng.randint(0, min(3, capacity - 1))
            chunk = rng.randint(1, min(3, capacity - sinks))
            c = _attention(None, kind, _log_int(rng, 1, 8), rng.choice([1, 2, 3, 5, 8, 12, 16]), rng.choice([64, 128, 128]),
                           _log_int(rng, 4, 30), _log_int(rng, 5, 52), capacity, sinks, chunk,
                           0 if kind in ("rollout", "prefill") else rng.randint(0, capacity + 4),
                           group=rng.choice([1, 1, 4]) if kind == "forward" else 1,
                           block=rng.choice([0, 0, 1]) if chunk > 1 and kind != "prefill" else 0,
                           relative=kind == "rollout" and rng.random() < 0.5,
                           chunks=rng.randint(2, 6) if kind in ("rollout", "prefill") else 1)
        w = work(c)
        if w["flops"] <= most and w["bytes"] <= most_bytes:
            return c


# ---- inputs ----------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, shape):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).to(torch.bfloat16)


def _attention_inputs(c, seed):
    """(history frames k, v [B, streamed*T, H, D], chunks): each chunk a tuple q, k, v, dout."""
    g = _generator(seed)
    T, H, D = c["grid_h"] * c["grid_w"], c["heads"], c["head_dim"]
    history = [_normal(g, (c["batch"], c["streamed"] * T, H, D)) for _ in range(2)]
    shape = (c["batch"] * c["group"], c["chunk"] * T, H, D)
    return history, [tuple(_normal(g, shape) for _ in range(4)) for _ in range(c["chunks"])]


def _loss_inputs(c, seed):
    g = _generator(seed)
    shape, n = (c["clips"], c["elems"]), c["clips"]
    x = [torch.randn(shape, generator=g, device=DEV) for _ in range(4)]
    x[0] = x[1] + 0.3 * x[0]  # the current policy stays near the old one, the reference nearer
    x[2] = x[1] + 0.1 * x[2]
    dtype = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    advantage = 1.5 * torch.randn(n, generator=g, device=DEV)
    mask = (torch.rand(n, generator=g, device=DEV) < 0.2).to(torch.int32)
    return [t.to(dtype) for t in x], advantage, mask


def _rope_pairs(D):
    s = D // 6
    return (D // 2 - 2 * s, s, s)


def prepare(case, seed):
    c = case
    if c["kind"] == "loss":
        x, advantage, mask = _loss_inputs(c, seed)
        return dict(kind="loss", x=x, advantage=advantage, mask=mask, loss=torch.empty(3, device=DEV),
                    grad=torch.empty(x[0].shape, dtype=torch.float32, device=DEV),
                    workspace=torch.empty(A.astro_nft_loss_workspace_bytes(*x[0].shape), dtype=torch.uint8, device=DEV))
    history, chunks = _attention_inputs(c, seed)
    T, n = c["grid_h"] * c["grid_w"], c["chunk"]
    cache = A.astro_kvcache_create(c["batch"], c["heads"], c["head_dim"], c["grid_h"], c["grid_w"], c["capacity"], c["sinks"],
                                   n, _rope_pairs(c["head_dim"]), ROPE_BASE, block_frames=c["block"],
                                   window_relative=c["relative"], reuse_staged=c["kind"] in ("update", "full"))
    for f in range(c["streamed"]):
        k, v = (x[:, f * T:(f + 1) * T].contiguous() for x in history)
        A.astro_kvcache_append(cache, k, v, 1)
    s = dict(kind=c["kind"], cache=cache, chunks=chunks, n=n, group=c["group"])
    if c["kind"] == "prefill":
        return s
    q = chunks[0][0]
    need = list(A.astro_group_attn_workspace_bytes(cache, n, c["group"]))
    if c["kind"] == "full":
        need.append(A.astro_chunk_attn_bwd_full_workspace_bytes(cache, n))
    # Two workspaces in turn, as for two layers or two steps in flight: a handle that may reuse staged
    # operands then stages those of every forward, and only the backward behind it picks them up.
    s["workspaces"] = [torch.empty(max(need), dtype=torch.uint8, device=DEV) for _ in range(2)]
    s["out"] = [torch.empty_like(q) for _ in chunks]
    s["lse"] = [torch.empty((q.shape[0], c["heads"], q.shape[1]), dtype=torch.float32, device=DEV) for _ in chunks]
    if c["kind"] in ("update", "full"):
        s["grads"] = [torch.empty(q.shape, dtype=torch.float32, device=DEV) for _ in range(3)]
    if c["kind"] == "full":
        ring = (c["batch"], c["capacity"] * T, c["heads"], c["head_dim"])
        s["ring_grads"] = [torch.zeros(ring, dtype=torch.float32, device=DEV) for _ in range(2)]
    return s


def _ring(cache):
    return [t.view(torch.bfloat16) for t in (cache.k_storage, cache.v_storage)]


def run(state):
    s = state
    if s["kind"] == "loss":
        A.astro_nft_loss(*s["x"], s["advantage"], s["mask"], A_MAX, BETA, LAMBDA_KL, s["loss"], s["grad"], s["workspace"])
        return [s["loss"], s["grad"]]
    cache, n = s["cache"], s["n"]
    if s["kind"] == "prefill":
        A.astro_kvcache_reset(cache)
        for _, k, v, _ in s["chunks"]:
            A.astro_kvcache_append(cache, k, v, n)
        return _ring(cache)
    workspace = s["workspaces"][0]
    s["workspaces"].reverse()
    if s["kind"] == "rollout":
        A.astro_kvcache_reset(cache)
        for (q, k, v, _), out, lse in zip(s["chunks"], s["out"], s["lse"]):
            A.astro_chunk_attn_fwd(cache, q, k, v, n, out, lse, workspace)
            A.astro_kvcache_append(cache, k, v, n)
        return s["out"] + s["lse"] + _ring(cache)
    (q, k, v, dout), out, lse = s["chunks"][0], s["out"][0], s["lse"][0]
    if s["group"] > 1:
        A.astro_group_attn_fwd(cache, q, k, v, n, s["group"], out, lse, workspace)
    else:
        A.astro_chunk_attn_fwd(cache, q, k, v, n, out, lse, workspace)
    if s["kind"] == "forward":
        return [out, lse]
    if s["kind"] == "update":
        A.astro_chunk_attn_bwd(cache, q, k, v, out, lse, dout, n, *s["grads"], workspace)
        return [out, lse] + s["grads"]
    A.astro_chunk_attn_bwd_full(cache, q, k, v, out, lse, dout, n, *s["grads"], *s["ring_grads"], workspace)
    return [out, lse] + s["grads"] + s["ring_grads"]


# ---- what a pass cannot do without -------------------------------------------------------------

def _resident(c, streamed):
    return min(streamed, c["capacity"])


def _chunk_pairs(c):
    """(query, key) pairs of one head inside a chunk."""
    T, n, b = c["grid_h"] * c["grid_w"], c["chunk"], c["block"] or c["chunk"]
    return T * T * sum(min(n, (f // b + 1) * b) for f in range(n))


def work(case):
    c = case
    if c["kind"] == "loss":
        n = c["clips"] * c["elems"]
        return {"bytes": n * (4 * (2 if c["dtype"] == "bf16" else 4) + 4), "flops": 20 * n}
    T, H, D, B = c["grid_h"] * c["grid_w"], c["heads"], c["head_dim"], c["batch"]
    candidates = B * c["group"]
    nq = c["chunk"] * T
    frame = T * H * D  # elements of one frame of one tensor
    chunk = candidates * c["chunk"] * frame
    if c["kind"] == "prefill":
        return {"bytes": c["chunks"] * 4 * chunk * 2, "flops": c["chunks"] * 3 * chunk}
    flops = nbytes = 0
    for i in range(c["chunks"]):
        resident = _resident(c, c["streamed"] + i * c["chunk"])
        ring_pairs, chunk_pairs = nq * resident * T, _chunk_pairs(c)
        per = D * H * candidates
        flops += 4 * (ring_pairs + chunk_pairs) * per
        nbytes += 2 * B * resident * frame * 2 + 4 * chunk * 2 + candidates * H * nq * 4  # ring, q k v out, lse
        if c["kind"] == "rollout":
            nbytes += 2 * chunk * 2  # ring rows written; k, v are read above
        if c["kind"] in ("update", "full"):
            flops += ((10 if c["kind"] == "full" else 6) * ring_pairs + 10 * chunk_pairs) * per
            nbytes += chunk * 2 + 3 * chunk * 4  # dout, three gradients
        if c["kind"] == "full":
            nbytes += 2 * B * resident * frame * 4
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # bf16 operands of every product (queries, keys, probabilities, dS) and bf16 outputs
    if case["kind"] == "loss":
        return {"rel": 1e-5}
    if case["kind"] == "prefill":
        return {"rel": 8e-3, "max": 3e-2}
    return {"rel": 1.5e-2, "max": 0.4}


# ---- the same in 64 bits -----------------------------------------------------------------------

def _rotate(c, x, position):
    """x [n_frames*T, H, D] in fp64, frame f at temporal position `position[f]`: adjacent pairs turned."""
    D = c["head_dim"]
    T = c["grid_h"] * c["grid_w"]
    token = torch.arange(x.shape[0], device=DEV)
    where = (torch.tensor(position, device=DEV, dtype=torch.float64)[token // T],
             (token % T // c["grid_w"]).double(), (token % c["grid_w"]).double())
    angle = torch.cat([p[:, None] * ROPE_BASE ** (-torch.arange(n, device=DEV, dtype=torch.float64) / n)
                       for p, n in zip(where, _rope_pairs(D))], dim=1)[:, None, :]
    a, b = x[..., 0::2], x[..., 1::2]
    cos, sin = angle.cos(), angle.sin()
    return torch.stack([a * cos - b * sin, a * sin + b * cos], dim=-1).flatten(-2)


def _rotate_back(c, x, position):
    """The transpose of _rotate."""
    swapped = torch.stack([x[..., 1::2], x[..., 0::2]], dim=-1).flatten(-2)
    y = _rotate(c, swapped, position)
    return torch.stack([y[..., 1::2], y[..., 0::2]], dim=-1).flatten(-2)


def _residents(c, streamed):
    """Frame numbers in the ring after `streamed` frames: sinks, then the window from old to new."""
    window = c["capacity"] - c["sinks"]
    sinks = list(range(min(c["sinks"], streamed)))
    return sinks + list(range(max(c["sinks"], streamed - window), streamed))


def _slot(c, n):
    return n if n < c["capacity"] else c["sinks"] + (n - c["sinks"]) % (c["capacity"] - c["sinks"])


def _positions(c, streamed):
    """Temporal positions of the residents and of the chunk's frames (as stored: only sinks move)."""
    moved = max(0, streamed - c["capacity"]) if c["relative"] else 0
    return ([f + moved if f < c["sinks"] else f for f in _residents(c, streamed)],
            list(range(streamed, streamed + c["chunk"])))


def _attend(c, q, k, v, kr, vr, dout=None):
    """One head: q, k, v [Nq, D] rotated chunk, kr, vr [Nr, D] residents.  out, lse and, with dout,
    dq, dk, dv over all visible keys (residents first)."""
    scale = 1.0 / math.sqrt(c["head_dim"])
    keys, values = torch.cat([kr, k]), torch.cat([vr, v])
    s = (q @ keys.T).mul_(scale)
    if c["block"]:
        rows = c["block"] * c["grid_h"] * c["grid_w"]
        block = torch.arange(q.shape[0], device=DEV) // rows
        s[:, kr.shape[0]:].masked_fill_(block[None, :] > block[:, None], -math.inf)
    lse = torch.logsumexp(s, dim=1)
    p = s.sub_(lse[:, None]).exp_()
    out = p @ values
    if dout is None:
        return out, lse
    dv = p.T @ dout
    ds = (dout @ values.T).sub_((dout * out).sum(1, keepdim=True)).mul_(p)
    return out, lse, (ds @ keys).mul_(scale), (ds.T @ q).mul_(scale), dv


def _exact_loss(c, seed):
    x, advantage, mask = _loss_inputs(c, seed)
    vt, vo, vr, tg = (t.double() for t in x)
    r = (advantage.double() / A_MAX).clamp(-1, 1)[:, None] * 0.5 + 0.5
    m = (mask != 0).double()[:, None]
    masked = float(m.sum())
    pos, neg, ref = (1 - BETA) * vo + BETA * vt - tg, (1 + BETA) * vo - BETA * vt - tg, vt - vr
    policy = (r * pos.square() + (1 - r) * neg.square()).sum() / c["clips"]
    kl = (m * ref.square()).sum() / masked if masked else torch.zeros((), device=DEV, dtype=torch.float64)
    grad = 2 * BETA / c["clips"] * (r * pos - (1 - r) * neg)
    if masked:
        grad = grad + 2 * LAMBDA_KL / masked * m * ref
    return [torch.stack([policy + LAMBDA_KL * kl, policy, kl]), grad]


def _exact_ring(c, frames):
    """Ring rows [B, H, C*T, D] after all frames were appended; slots never written are zero."""
    T, D = c["grid_h"] * c["grid_w"], c["head_dim"]
    streamed = frames[0].shape[1] // T
    ring = [torch.zeros(c["batch"], c["heads"], c["capacity"] * T, D, device=DEV, dtype=torch.float64) for _ in range(2)]
    position = dict(zip(_residents(c, streamed), _positions(c, streamed)[0]))
    for b in range(c["batch"]):
        for f, at in position.items():
            rows = slice(_slot(c, f) * T, (_slot(c, f) + 1) * T)
            k, v = (x[b, f * T:(f + 1) * T].double() for x in frames)
            ring[0][b, :, rows] = _rotate(c, k, [at]).transpose(0, 1)
            ring[1][b, :, rows] = v.transpose(0, 1)
    return [x.flatten() for x in ring]


def exact(case, seed):
    c = case
    if c["kind"] == "loss":
        return _exact_loss(c, seed)
    history, chunks = _attention_inputs(c, seed)
    T, H, D, G = c["grid_h"] * c["grid_w"], c["heads"], c["head_dim"], c["group"]
    if c["kind"] in ("rollout", "prefill"):  # every chunk becomes history of the next
        frames = [torch.cat([x[i] for x in chunks], dim=1) for i in (1, 2)]
    else:
        frames = history
    if c["kind"] == "prefill":
        return _exact_ring(c, frames)
    new = lambda *shape: torch.zeros(shape, device=DEV, dtype=torch.float64)
    outs, lses = [], []
    nq = c["chunk"] * T
    grads = c["kind"] in ("update", "full")
    if grads:
        dq, dk, dv = (new(c["batch"], nq, H, D) for _ in range(3))
        ring = [new(c["batch"], c["capacity"] * T, H, D) for _ in range(2 if c["kind"] == "full" else 0)]
    for i, (q, k, v, dout) in enumerate(chunks):
        streamed = c["streamed"] + i * c["chunk"]
        residents, (ring_pos, chunk_pos) = _residents(c, streamed), _positions(c, streamed)
        out, lse = new(*q.shape), new(q.shape[0], H, nq)
        for b in range(c["batch"]):
            token = torch.cat([torch.arange(f * T, (f + 1) * T, device=DEV) for f in residents] or
                              [torch.zeros(0, device=DEV, dtype=torch.long)])
            kr, vr = (x[b, token].double() for x in frames)
            kr = _rotate(c, kr, ring_pos) if residents else kr
            for a in range(b * G, (b + 1) * G):
                qa, ka, va = _rotate(c, q[a].double(), chunk_pos), _rotate(c, k[a].double(), chunk_pos), v[a].double()
                got_q, got_k, got_v = ([], [], [])
                for h in range(H):
                    r = _attend(c, qa[:, h], ka[:, h], va[:, h], kr[:, h], vr[:, h], dout[a, :, h].double() if grads else None)
                    out[a, :, h], lse[a, h] = r[0], r[1]
                    if grads:
                        got_q.append(r[2]); got_k.append(r[3]); got_v.append(r[4])
                if grads:
                    n_ring = token.numel()
                    gk, gv = torch.stack(got_k, 1), torch.stack(got_v, 1)
                    dq[a] = _rotate_back(c, torch.stack(got_q, 1), chunk_pos)
                    dk[a], dv[a] = _rotate_back(c, gk[n_ring:], chunk_pos), gv[n_ring:]
                    if c["kind"] == "full" and residents:
                        row = torch.cat([torch.arange(_slot(c, f) * T, (_slot(c, f) + 1) * T, device=DEV) for f in residents])
                        ring[0][b, row], ring[1][b, row] = _rotate_back(c, gk[:n_ring], ring_pos), gv[:n_ring]
        outs.append(out)
        lses.append(lse)
    if c["kind"] == "rollout":
        return outs + lses + _exact_ring(c, frames)
    return outs + lses + ([dq, dk, dv] + ring if grads else [])

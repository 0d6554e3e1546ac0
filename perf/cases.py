"""The work a program has this library do, as measurable cases.

A program that generates video holds, per layer, a ring of cached tokens. For every chunk of
new frames and every denoising step it writes the chunk's tokens into the ring (`write`) and
attends the chunk's queries over the window (`attend`), one after the other (`step`), or runs the
whole attention layer on the chunk (`layer`). The dense per-head cache that the latent cache
replaces has its own write and attention (`dense_write`, `dense_attend`), which the rollout
comparison runs at the same shapes. Shapes are those of the Wan2.1-1.3B layer and of the tiny and
small test layers, plus the range between them: latent widths of the d_c sweep, windows that are
still filling, windows with a sink frame, chunks of one to three frames, blocks of a few query
tokens per video, and batches.

Every case is a dict of plain values:
  op                       step | write | attend | layer | dense_write | dense_attend
  d_model .. d_v, grid_*   the layer's shapes (videomla_dims)
  window, chunk, sink      frames held, frames per call, sink frames
  split                    RoPE channel split: wan (8, 4, 4 pairs), paper (6, 5, 5 with Wan's
                           bands) or tiny (2, 1, 1)
  frame_end, batch         first frame of the chunk; videos
  q_begin, q_count         block of the chunk's query tokens (q_count 0: the whole chunk)
  form                     latent, or auto (the faster of the two exact forms)
  gain                     factor on the queries (1: flat softmax, 4: peaked)
  d_q                      query latent width (layer)
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import torch

import paper_2605_30351_amd as vm

BF16 = torch.bfloat16

_WAN = dict(d_model=1536, n_heads=12, d_nope=128, d_rope=32, d_c=192, d_v=128, grid_h=30, grid_w=52,
            window=21, chunk=3, sink=0, split="wan", frame_end=24, batch=1, q_begin=0, q_count=0,
            form="latent", gain=1.0, d_q=0)
_SMALL = dict(_WAN, d_model=256, n_heads=2, grid_h=6, grid_w=10, window=5, chunk=2, frame_end=8)
_TINY = dict(_WAN, d_model=64, n_heads=2, d_nope=32, d_rope=8, d_c=16, d_v=32, grid_h=4, grid_w=4,
             window=3, chunk=1, split="tiny", frame_end=5)


def listed():
    """The listed cases, smallest first."""
    def case(name, base, op, **kw):
        return dict(base, name=name, op=op, **kw)
    return [
        # the smallest call: the tiny test layer's write and attend, where latency is everything
        case("tiny-step", _TINY, "step"),
        # a small layer, three videos, a ragged last key tile and a window still filling
        case("small-attend-b3", _SMALL, "attend", batch=3, frame_end=2, gain=4.0),
        # one Wan layer's cache write of a 3-frame chunk, for one video ...
        case("wan-write-b1", _WAN, "write"),
        # ... and for the four videos of a batched rollout
        case("wan-write-b4", _WAN, "write", batch=4),
        # a block of 16 query tokens per video over the full window: bandwidth-bound decode
        case("wan-few-query-b8", _WAN, "attend", batch=8, q_begin=100, q_count=16),
        # long rollout: one sink frame and the six most recent frames
        case("wan-sink-attend", _WAN, "attend", window=7, sink=1, frame_end=237),
        # the headline: one layer's denoising step, write and attend over the full window
        case("wan-step", _WAN, "step"),
        # the whole layer, from the chunk's input to the output projection
        case("wan-layer", _WAN, "layer", d_q=768),
        # the paper's head split with the form left to the library
        case("wan-auto-attend", _WAN, "attend", d_nope=96, split="paper", form="auto"),
        # the widest latent of the d_c sweep
        case("wan-dc512-attend", _WAN, "attend", d_c=512),
        # the dense comparator's cache write in the batched rollout
        case("wan-dense-write-b4", _WAN, "dense_write", batch=4),
        # the dense comparator's attention over the full window
        case("wan-dense-attend", _WAN, "dense_attend"),
    ]


# A drawn case costs no more than this many multiply-add FLOPs and bytes: the widest-latent
# listed case is 4e12 FLOPs at a third of the rate that the others reach.
_MAX_FLOPS, _MAX_BYTES = 1.8e12, 1.5e9


def draw(rng):
    """One more case of the same ranges."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    while True:
        op = rng.choice(["step", "write", "attend", "attend", "attend", "layer", "dense_write",
                         "dense_attend"])
        if rng.random() < 0.12:  # layers of the tiny and small test shapes
            c = dict(rng.choice([_TINY, _SMALL]), grid_h=rng.randint(3, 12), grid_w=rng.randint(3, 12))
            if c["d_c"] == 16 and op.startswith("dense"):
                continue  # the dense comparator is built for 128-wide heads
        else:
            c = dict(_WAN, grid_h=log_int(6, 30), grid_w=log_int(8, 52))
            c["d_c"] = rng.choice([64, 128, 192, 192, 192, 192, 256, 512])
            c["n_heads"] = rng.choice([12, 12, 12, 8, 16])
            c["d_model"] = rng.choice([1536, 1536, 1536, 1024, 768])
            if rng.random() < 0.4:
                c.update(d_nope=96, split="paper")
            c["window"] = rng.randint(6, 21)
            c["chunk"] = rng.randint(1, 3)
        c["op"] = op
        if not op.startswith("dense") and rng.random() < 0.2 and c["window"] - 1 >= c["chunk"]:
            c["sink"] = 1
        # a third of the calls come while the window is still filling
        c["frame_end"] = rng.randint(0, 2 if rng.random() < 1 / 3 else 3 * c["window"])
        c["batch"] = rng.choice([1, 1, 1, 2, 3, 4, 8])
        c["gain"] = rng.choice([1.0, 1.0, 4.0])
        if op in ("attend", "dense_attend") and rng.random() < 0.4:
            tokens = c["chunk"] * c["grid_h"] * c["grid_w"]
            c["q_count"] = min(tokens, log_int(1, 400))
            c["q_begin"] = rng.randint(0, tokens - c["q_count"])
        if op == "attend" and rng.random() < 0.3:
            c["form"] = "auto"
        if op == "layer":
            c["d_q"] = rng.choice([768, 768, 512, 1000, 384])
        w = work(c)
        if w["flops"] <= _MAX_FLOPS and w["bytes"] <= _MAX_BYTES:
            return c


# ---- shapes ---------------------------------------------------------------------------------

_PAIRS = {"wan": ((8, 4, 4), (0, 0, 0)), "paper": ((6, 5, 5), (44, 42, 42)),
          "tiny": ((2, 1, 1), (0, 0, 0))}


def _dims(c):
    pairs, bands = _PAIRS[c["split"]]
    return SimpleNamespace(
        d_model=c["d_model"], n_heads=c["n_heads"], d_nope=c["d_nope"], d_rope=c["d_rope"],
        d_c=c["d_c"], d_v=c["d_v"], grid_h=c["grid_h"], grid_w=c["grid_w"],
        window_frames=c["window"], chunk_frames=c["chunk"], rope_pairs=pairs, rope_band_dim=bands,
        rope_base=10000.0, softmax_scale=0.0, kv_norm_eps=1e-6, sink_frames=c["sink"])


def _hw(c):
    return c["grid_h"] * c["grid_w"]


def _n_chunk(c):
    return c["chunk"] * _hw(c)


def _n_query(c):
    return c["q_count"] or _n_chunk(c) - c["q_begin"]


def _n_valid(c):
    return min(c["window"], c["frame_end"] + c["chunk"]) * _hw(c)


def work(case):
    c = case
    B, H, S, Nq, M = c["batch"], c["n_heads"], _n_valid(c), _n_query(c), c["batch"] * _n_chunk(c)
    dm, dn, dr, dc, dv = c["d_model"], c["d_nope"], c["d_rope"], c["d_c"], c["d_v"]
    rows = B * Nq * H
    ring = B * S * (dc + dr) * 2
    w_write = {"bytes": M * (dm + dc + dr) * 2 + (dc + dr) * dm * 2 + _n_chunk(c) * 4,
               "flops": 2 * M * (dc + dr) * dm}
    latent = 2 * rows * (dn * dc + dc * dv) + 2 * rows * S * (2 * dc + dr)
    per_head = 2 * B * S * H * dc * (dn + dv) + 2 * rows * S * (dn + dr + dv)
    w_attend = {"bytes": rows * (dn + dr + dv) * 2 + ring + H * (dn + dv) * dc * 2,
                "flops": min(latent, per_head) if c["form"] == "auto" else latent}
    op = c["op"]
    if op == "write":
        return w_write
    if op == "attend":
        return w_attend
    if op == "step":  # the chunk's own ring rows are written once and read once
        return {k: w_write[k] + w_attend[k] for k in w_write}
    if op == "layer":
        dq = c["d_q"]
        weights = dq * dm + H * (dc + dr) * dq + dm * H * dc
        return {"bytes": 2 * B * Nq * dm * 2 + ring + weights * 2,
                "flops": 2 * B * Nq * weights + 2 * rows * S * (2 * dc + dr)}
    if op == "dense_write":
        return {"bytes": M * dm * 2 + 2 * H * dv * dm * 2 + M * H * 2 * dv * 2 + _n_chunk(c) * 4,
                "flops": 2 * M * 2 * H * dv * dm}
    return {"bytes": rows * 2 * dv * 2 + B * S * H * 2 * dv * 2, "flops": 2 * rows * S * 2 * dv}


def tolerance(case):
    """bf16 operands and results with fp32 sums: the relative error is that of the bf16 roundings
    on the way (q_cat, the probabilities, o_lat and the output; for the layer also its inner
    activations). Against 64 bits: 0.0017 for the writes, 0.0023 to 0.0048 for the attention
    (the more peaked the softmax, the larger); about four times that is allowed, and one value
    may be off by a few bf16 steps."""
    if case["op"] in ("write", "dense_write"):
        return {"rel": 7e-3, "max": 0.03}
    return {"rel": 2e-2, "max": 0.1}


# ---- inputs ---------------------------------------------------------------------------------

def _inputs(c, seed):
    """Seeded inputs on the GPU: activations N(0, 1), weights N(0, 1 / fan_in), latents of unit
    RMS as the cache's norm leaves them, all bf16."""
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, std=1.0):
        return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0, std, generator=gen).to(BF16)

    B, H, Nq = c["batch"], c["n_heads"], _n_query(c)
    dm, dn, dr, dc, dv = c["d_model"], c["d_nope"], c["d_rope"], c["d_c"], c["d_v"]
    ring = c["window"] * _hw(c)
    op = c["op"]
    t = {}
    if op in ("step", "write"):
        t["x"] = normal(B, _n_chunk(c), dm)
        t["w_dkv"] = normal(dc, dm, std=dm ** -0.5)
        t["w_kr"] = normal(dr, dm, std=dm ** -0.5)
        t["gamma"] = (0.5 + torch.rand(dc, generator=gen, device="cuda")).to(BF16)
    if op in ("step", "attend", "layer"):
        t["c_kv"] = normal(B, ring, dc)
        t["k_r"] = normal(B, ring, dr)
        t["w_uk"] = normal(H * dn, dc, std=dc ** -0.5)
        t["w_uv"] = normal(H * dv, dc, std=dc ** -0.5)
    if op in ("step", "attend"):
        t["q_nope"] = normal(B, Nq, H, dn, std=c["gain"])
        t["q_r"] = normal(B, Nq, H, dr, std=c["gain"])
    if op == "layer":
        dq = c["d_q"]
        t["x"] = normal(B, Nq, dm)
        t["w_dq"] = normal(dq, dm, std=dm ** -0.5)
        t["gamma_q"] = (0.5 + torch.rand(dq, generator=gen, device="cuda")).to(BF16)
        t["w_uq"] = normal(H * dn, dq, std=c["gain"] * dq ** -0.5)
        t["w_qr"] = normal(H * dr, dq, std=c["gain"] * dq ** -0.5)
        t["w_o"] = normal(dm, H * dv, std=(H * dv) ** -0.5)
    if op == "dense_write":
        t["x"] = normal(B, _n_chunk(c), dm)
        t["w_k"] = normal(H * dv, dm, std=dm ** -0.5)
        t["w_v"] = normal(H * dv, dm, std=dm ** -0.5)
    if op == "dense_attend":
        t["kv"] = normal(B, ring, H, 2 * dv)
        t["q"] = normal(B, Nq, H, dv, std=c["gain"])
    return t


def prepare(case, seed):
    c, d = case, _dims(case)
    t = _inputs(c, seed)
    B, H, Nq, ring = c["batch"], c["n_heads"], _n_query(c), c["window"] * _hw(c)
    s = SimpleNamespace(op=c["op"], d=d, fe=c["frame_end"], batch=B, d_q=c["d_q"], **t)
    # the write cases fill a fresh ring; a step's ring holds the earlier frames
    if c["op"] == "write":
        s.c_kv = torch.zeros(B, ring, c["d_c"], dtype=BF16, device="cuda")
        s.k_r = torch.zeros(B, ring, c["d_rope"], dtype=BF16, device="cuda")
    if c["op"] in ("step", "write"):  # packed once, at model load
        s.panel = torch.empty(vm.write_weights_bytes(d), dtype=torch.uint8, device="cuda")
        vm.prepare_write_weights(d, s.w_dkv, s.w_kr, s.panel)
    if c["op"] in ("step", "write", "dense_write"):
        s.slots = torch.empty(_n_chunk(c), dtype=torch.int32, device="cuda")
    if c["op"] == "dense_write":
        s.kv = torch.zeros(B, ring, H, 2 * c["d_v"], dtype=BF16, device="cuda")
    if c["op"] in ("attend", "step", "layer", "dense_attend"):
        plain = not c["q_begin"] and not c["q_count"] and c["form"] == "latent"
        s.opts = None if plain else vm.AttendOpts(form=c["form"], query_begin=c["q_begin"],
                                                  query_count=c["q_count"])
        if c["op"] == "layer":
            s.weights = torch.empty(vm.layer_weights_bytes(d, c["d_q"]), dtype=torch.uint8, device="cuda")
            vm.prepare_layer_weights(d, c["d_q"], s.w_dq, s.gamma_q, s.w_uq, s.w_qr, s.w_uk, s.w_uv,
                                     s.w_o, s.weights)
            nbytes = vm.attend_layer_workspace_bytes(d, c["d_q"], B, s.opts)
            s.out = torch.empty(B, Nq, c["d_model"], dtype=BF16, device="cuda")
        elif c["op"] == "dense_attend":
            nbytes = vm.dense_attend_workspace_bytes(d, B, s.opts)
            s.out = torch.empty(B, Nq, H, c["d_v"], dtype=BF16, device="cuda")
        else:
            nbytes = vm.attend_workspace_bytes(d, B, s.opts)
            s.out = torch.empty(B, Nq, H, c["d_v"], dtype=BF16, device="cuda")
        s.workspace = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    return s


def run(state):
    s = state
    if s.op in ("step", "write"):
        vm.cache_write_prepared(s.d, s.fe, s.batch, s.x, s.panel, s.gamma, s.c_kv, s.k_r, s.slots)
    if s.op in ("step", "attend"):
        vm.attend(s.d, s.fe, s.batch, s.q_nope, s.q_r, s.w_uk, s.w_uv, s.c_kv, s.k_r, s.out,
                  s.workspace, opts=s.opts)
    if s.op == "layer":
        vm.attend_layer(s.d, s.fe, s.batch, s.d_q, s.x, s.weights, s.c_kv, s.k_r, s.out,
                        s.workspace, opts=s.opts)
    if s.op == "dense_write":
        vm.dense_cache_write(s.d, s.fe, s.batch, s.x, s.w_k, s.w_v, s.kv, s.slots)
    if s.op == "dense_attend":
        vm.dense_attend(s.d, s.fe, s.batch, s.q, s.kv, s.out, s.workspace, opts=s.opts)
    if s.op == "write":
        return s.c_kv, s.k_r, s.slots
    if s.op == "step":
        return s.out, s.c_kv, s.k_r, s.slots
    if s.op == "dense_write":
        return s.kv, s.slots
    return s.out


# ---- the same in 64 bits, plain torch ---------------------------------------------------------

def _rope_table(split, d_rope):
    """Axis (0 frame, 1 row, 2 column) and frequency of every interleaved channel pair."""
    if split == "head":  # the dense comparator's full head
        k = d_rope // 6
        bands = (d_rope - 4 * k, 2 * k, 2 * k)
        pairs = tuple(b // 2 for b in bands)
    else:
        pairs, bands = _PAIRS[split]
    axis, theta = [], []
    for a in range(3):
        for k in range(pairs[a]):
            axis.append(a)
            theta.append(10000.0 ** (-2.0 * k / (bands[a] or 2 * pairs[a])))
    return torch.tensor(axis, device="cuda"), torch.tensor(theta, dtype=torch.float64, device="cuda")


def _rotate(v, pos, split):
    """v [..., n, (heads,) d] rotated; pos [n, 3] per token; heads where v has one axis more."""
    axis, theta = _rope_table(split, v.shape[-1])
    ang = pos.double()[:, axis] * theta
    cos, sin = torch.cos(ang), torch.sin(ang)
    if v.dim() == 4:
        cos, sin = cos[:, None], sin[:, None]
    a, b = v[..., 0::2], v[..., 1::2]
    return torch.stack((a * cos - b * sin, a * sin + b * cos), -1).flatten(-2)


def _grid_pos(c, frames):
    """(frame, row, column) of every token of the given frame numbers, in order."""
    f = torch.as_tensor(frames, device="cuda").repeat_interleave(_hw(c))
    r = torch.arange(_hw(c), device="cuda").repeat(len(frames))
    return torch.stack((f, r // c["grid_w"], r % c["grid_w"]), -1)


def _frame_slot(c, f):
    S = c["sink"]
    return f if f < S else S + (f - S) % (c["window"] - S)


def _chunk_frames(c):
    return list(range(c["frame_end"], c["frame_end"] + c["chunk"]))


def _ring_rows(c):
    """Ring row of every token of the chunk."""
    base = torch.tensor([_frame_slot(c, f) * _hw(c) for f in _chunk_frames(c)], device="cuda")
    return (base[:, None] + torch.arange(_hw(c), device="cuda")).flatten()


def _local_lo(c):
    hi = c["frame_end"] + c["chunk"]
    return max(c["sink"], hi - (c["window"] - c["sink"]))


def _query_pos(c):
    frames = _chunk_frames(c)
    if c["sink"]:
        frames = [f if f < c["sink"] else c["sink"] + f - _local_lo(c) for f in frames]
    return _grid_pos(c, frames)[c["q_begin"]:c["q_begin"] + _n_query(c)]


def _window_keys(c, k_r):
    """Positional keys of the valid slots as the scores see them (rotated now with a sink)."""
    k = k_r[:, :_n_valid(c)]
    if not c["sink"]:
        return k
    S, L = c["sink"], c["window"] - c["sink"]
    frames = []
    for fs in range(_n_valid(c) // _hw(c)):
        frames.append(fs if fs < S else S + ((fs - S) - (_local_lo(c) - S)) % L)
    return _rotate(k, _grid_pos(c, frames), c["split"])


def _softmax_mix(q, k, v, scale):
    """softmax(scale q k^T) v for one batch element and head group: q [R, d], k [S, d], v [S, e]."""
    out = torch.empty(q.shape[0], v.shape[1], dtype=torch.float64, device="cuda")
    step = max(1, (1 << 27) // k.shape[0])
    kt = k.t().contiguous()
    for r in range(0, q.shape[0], step):
        p = torch.softmax((q[r:r + step] @ kt) * scale, -1)
        out[r:r + step] = p @ v
    return out


def _latent_mix(c, q_nope, q_r, t, c_kv, keys):
    """o_lat [B, Nq, H, d_c] of 64-bit queries (q_r already rotated) over the window."""
    B, Nq, H, dn = q_nope.shape
    w_uk = t["w_uk"].double().view(H, dn, c["d_c"])
    scale = (dn + c["d_rope"]) ** -0.5
    q_lat = torch.stack([q_nope[:, :, h] @ w_uk[h] for h in range(H)], 2)
    q = torch.cat((q_lat, q_r), -1)
    res = []
    for b in range(B):
        lat = c_kv[b, :_n_valid(c)]
        res.append(_softmax_mix(q[b].reshape(Nq * H, -1), torch.cat((lat, keys[b]), -1), lat, scale))
    return torch.stack(res).view(B, Nq, H, c["d_c"])


def _per_head(o_lat, w_uv, d_v):
    H = o_lat.shape[2]
    w = w_uv.double().view(H, d_v, -1)
    return torch.stack([o_lat[:, :, h] @ w[h].t() for h in range(H)], 2)


def exact(case, seed):
    c = case
    t = _inputs(c, seed)
    dr, dc, dv, H = c["d_rope"], c["d_c"], c["d_v"], c["n_heads"]
    op = c["op"]
    if op in ("step", "write"):
        x = t["x"].double()
        lat = x @ t["w_dkv"].double().t()
        lat = lat * torch.rsqrt((lat * lat).mean(-1, keepdim=True) + 1e-6) * t["gamma"].double()
        key = x @ t["w_kr"].double().t()
        if not c["sink"]:
            key = _rotate(key, _grid_pos(c, _chunk_frames(c)), c["split"])
        rows = _ring_rows(c)
        if op == "write":
            ring = c["window"] * _hw(c)
            c_kv = torch.zeros(c["batch"], ring, dc, dtype=torch.float64, device="cuda")
            k_r = torch.zeros(c["batch"], ring, dr, dtype=torch.float64, device="cuda")
        else:
            c_kv, k_r = t["c_kv"].double(), t["k_r"].double()
        c_kv[:, rows], k_r[:, rows] = lat, key
        if op == "write":
            return c_kv, k_r, rows.to(torch.int32)
    if op in ("attend", "layer"):
        c_kv, k_r = t["c_kv"].double(), t["k_r"].double()
    if op in ("step", "attend"):
        q_r = _rotate(t["q_r"].double(), _query_pos(c), c["split"])
        o_lat = _latent_mix(c, t["q_nope"].double(), q_r, t, c_kv, _window_keys(c, k_r))
        out = _per_head(o_lat, t["w_uv"], dv)
        return out if op == "attend" else (out, c_kv, k_r, rows.to(torch.int32))
    if op == "layer":
        u = t["x"].double() @ t["w_dq"].double().t()
        cq = u * torch.rsqrt((u * u).mean(-1, keepdim=True) + 1e-6) * t["gamma_q"].double()
        q_nope = (cq @ t["w_uq"].double().t()).unflatten(-1, (H, -1))
        q_r = (cq @ t["w_qr"].double().t()).unflatten(-1, (H, -1))
        o_lat = _latent_mix(c, q_nope, _rotate(q_r, _query_pos(c), c["split"]), t, c_kv,
                            _window_keys(c, k_r))
        return _per_head(o_lat, t["w_uv"], dv).flatten(-2) @ t["w_o"].double().t()
    if op == "dense_write":
        x = t["x"].double()
        k = (x @ t["w_k"].double().t()).unflatten(-1, (H, dv))
        v = (x @ t["w_v"].double().t()).unflatten(-1, (H, dv))
        kv = torch.zeros(c["batch"], c["window"] * _hw(c), H, 2 * dv, dtype=torch.float64, device="cuda")
        rows = _ring_rows(c)
        kv[:, rows] = torch.cat((_rotate(k, _grid_pos(c, _chunk_frames(c)), "head"), v), -1)
        return kv, rows.to(torch.int32)
    q = _rotate(t["q"].double(), _query_pos(c), "head")
    out = torch.empty_like(q)
    for b in range(c["batch"]):
        for h in range(H):
            kv = t["kv"][b, :_n_valid(c), h].double()
            out[b, :, h] = _softmax_mix(q[b, :, h], kv[:, :dv], kv[:, dv:], dv ** -0.5)
    return out

"""What the framework's users have it do, as measurable cases.

A case is one pass through the public entry points over a synthetic stream: whole per-chunk
steps (score, select, compact, attend), the planners, the compactions, chunk attention, decode
attention and the native (logical-only) layout, from the 1.6K-token test stream up to 36 layers
of a 32K-token history.  Structure (units, holes, plans) follows from the case alone; keys,
values and queries are drawn on the GPU from the seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2609_34653_amd import omnitide as ot
from paper_2609_34653_amd.step import StreamStep

SYS, VIDEO, AUDIO, TEXT, MARK = 0, 1, 2, 3, 4
WEIGHTS = (2.0, 1.0, 1.5, 2.0)
ROPE_BASE = 1.0e6
MAX_UNITS = 8192


# ------------------------------------------------------------------------------------- cases

def listed():
    return [
        # The smallest stream of the tests (float32 pool, 1.6K tokens): what the four calls of
        # a step cost when there is next to nothing to compute.
        dict(name="step_tiny_1p6k_f32", kind="step", layers=1, slots=1634, frame=64, every=1,
             sys=0, holes=0.0, chunk=89, budget=512, hq=4, hkv=1, d=64, f32=True),
        # The benchmark's step: one layer of an 80K-token history with holes, 665-token chunk.
        dict(name="step_history_80k", kind="step", layers=1, slots=81920, frame=640, every=5,
             sys=0, holes=0.3, chunk=665, budget=16384, hq=32, hkv=8, d=128, f32=False),
        # All 36 layers of a high-resolution 32K-token history as one call of each entry point.
        dict(name="step_hires_32k_36layer", kind="step", layers=36, slots=32768, frame=2304,
             every=1, sys=0, holes=0.0, chunk=2329, budget=8192, hq=32, hkv=8, d=128, f32=False),
        # Score and selection of a long talk: an hour and more of one-second audio units and
        # text turns with few frames, so thousands of short units compete for the budget.
        dict(name="plan_talk_many_units", kind="plan", layers=1, slots=120000, frame=64,
             every=20, sys=96, holes=0.1, chunk=89, budget=16384, hq=32, hkv=8, d=128, f32=False),
        # The span plan (sink prefixes, text budget, trimming) of the 80K history in grammar
        # units, then its compaction with rotary re-encoding of the moved keys.
        dict(name="spans_rope_80k", kind="spans", layers=1, slots=81920, frame=640, every=5,
             sys=64, holes=0.3, chunk=665, budget=16384, hq=32, hkv=8, d=128, f32=False,
             rope=128, half=True),
        # Compaction with the interleaved pairing over a float32 pool, two layers, partial
        # rotary width: the other type and pairing that the calls offer.
        dict(name="compact_rope_f32_2x12k", kind="compact", layers=2, slots=12345, frame=640,
             every=1, sys=33, holes=0.1, chunk=201, budget=6144, hq=16, hkv=4, d=128, f32=True,
             rope=64, half=False),
        # One layer's chunk attention over the 8K stream's compacted history, bf16 output (a
        # model that keeps its activations in bf16).
        dict(name="attn_4k_bf16_out", kind="attn", layers=1, ctx=4761, cap=4761, chunk=665,
             hq=32, hkv=8, d=128, f32=False, out_bf16=True),
        # Chunk attention over a float32 pool of a small model (d = 64), ragged sizes.
        dict(name="attn_11k_f32_d64", kind="attn", layers=1, ctx=11003, cap=12288, chunk=331,
             hq=14, hkv=2, d=64, f32=True, out_bf16=False),
        # Decode of one token over one layer's compacted 80K history.
        dict(name="decode_17k", kind="decode", layers=1, ctx=16948, cap=17049, nq=1, hq=32,
             hkv=8, d=128),
        # Decode of two tokens (a drafted one beside the last) for 24 streams at once.
        dict(name="decode_24x9k_2tok", kind="decode", layers=24, ctx=9173, cap=10521, nq=2,
             hq=32, hkv=8, d=128),
        # The native layout's step over the 80K pool: logical eviction, the chunk into the
        # lowest holes, attention in position order.
        dict(name="native_80k_position_order", kind="native", layers=1, slots=98304, frame=640,
             every=5, sys=0, holes=0.3, chunk=665, budget=16384, hq=32, hkv=8, d=128,
             traversal=2, pack=0),
        # Decode over a native pool's physical span with tile skipping.
        dict(name="decode_native_38k_skip", kind="decode_span", layers=1, slots=37997, frame=640,
             every=1, sys=0, holes=0.5, nq=1, hq=32, hkv=8, d=128, traversal=1),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_HEADS = [(4, 1, 64), (14, 2, 64), (16, 4, 128), (16, 2, 128), (28, 4, 128), (32, 8, 128),
          (32, 8, 128), (8, 8, 64)]


def draw(rng):
    kind = rng.choice(["step", "step", "plan", "spans", "compact", "attn", "attn", "decode",
                       "native", "span_attn", "decode_span"])
    hq, hkv, d = rng.choice(_HEADS)
    c = dict(kind=kind, hq=hq, hkv=hkv, d=d)
    layers = _log(rng, 1, 24)
    if kind in ("step", "plan", "spans", "compact"):
        slots = _log(rng, 1500, min(120000, 600000 // layers))
        if kind == "plan":
            frame, every = rng.choice([(64, 1), (64, 20), (576, 10), (640, 5)])
        else:
            frame, every = rng.choice([(64, 1), (576, 2), (640, 1), (640, 5), (2304, 4)])
        chunk = min(_log(rng, 17, 2400), slots)
        c.update(layers=layers, slots=slots, frame=frame, every=every,
                 sys=rng.choice([0, 33, 64]), holes=round(rng.uniform(0.0, 0.4), 2),
                 chunk=chunk, budget=max(96, int(slots * rng.uniform(0.15, 0.6))),
                 f32=rng.random() < 0.25)
        if kind in ("spans", "compact"):
            c.update(rope=rng.choice([0, 32, 64, d]), half=rng.random() < 0.6)
    elif kind == "attn":
        ctx = _log(rng, 600, 40000)
        c.update(layers=_log(rng, 1, 8), ctx=ctx, cap=ctx + rng.randint(0, 1500),
                 chunk=min(_log(rng, 16, 2400), ctx), f32=rng.random() < 0.3,
                 out_bf16=rng.random() < 0.5)
    elif kind == "decode":
        ctx = _log(rng, 400, 60000)
        c.update(layers=_log(rng, 1, 36), ctx=ctx, cap=ctx + rng.randint(0, 3000),
                 nq=rng.randint(1, max(1, 8 // (hq // hkv))))
    else:
        slots = _log(rng, 4000, 90000)
        c.update(layers=_log(rng, 1, 6), slots=slots, frame=rng.choice([64, 640, 2304]),
                 every=rng.choice([1, 2, 5]), sys=0, holes=round(rng.uniform(0.1, 0.6), 2),
                 traversal=rng.choice([0, 1, 1, 2, 2]))
        if kind == "native":
            c.update(chunk=_log(rng, 17, 1200), budget=max(96, int(slots * rng.uniform(0.15, 0.5))),
                     pack=rng.choice([0, 0, 1, 8]))
        elif kind == "span_attn":
            c.update(chunk=_log(rng, 17, 1200))
        else:
            c.update(nq=rng.randint(1, max(1, 8 // (hq // hkv))))
    return c


# --------------------------------------------------------------------------------- structure

def _units(c, grammar=False):
    """History units as (per-slot modality tags) arrays adding up to c["slots"] slots: a frame
    every `every` seconds, 25 audio tokens a second, a text turn of 16 to 64 tokens now and
    then, behind a system prefix of `sys` tokens.  Grammar units hold a second's frame, audio and
    text between structural markers."""
    rng = random.Random(1000003 * c["slots"] + 31 * c["frame"] + c["every"])
    units, n, sec = [], 0, 0
    if c["sys"]:
        units.append([SYS] * c["sys"])
        n += c["sys"]
    while n < c["slots"]:
        parts = []
        if sec % c["every"] == 0:
            parts.append((VIDEO, c["frame"]))
        parts.append((AUDIO, 25))
        if rng.random() < 0.1:
            parts.append((TEXT, rng.randint(16, 64)))
        if grammar:
            u = [MARK]
            for m, k in parts:
                u += [m] * k if m == TEXT else [MARK] + [m] * k + [MARK]
            new = [u + [MARK]]
        else:
            new = [[m] * k for m, k in parts]
        for u in new:
            u = u[:c["slots"] - n]
            if u and len(units) == MAX_UNITS:       # the rest goes into the last unit
                units[-1] = units[-1] + u
            elif u:
                units.append(u)
            n += len(u)
        sec += 1
    return units


class Layout:
    """Tags of the history pool, units evicted earlier left as holes (the newest are whole)."""

    def __init__(self, c, grammar=False):
        units = _units(c, grammar)
        rng = random.Random(7 * c["slots"] + int(100 * c["holes"]))
        recent = max(1, len(units) // 20)
        lens = np.array([len(u) for u in units])
        gone = np.array([0 < i < len(units) - recent and rng.random() < c["holes"]
                         for i in range(len(units))])
        self.modality = np.concatenate([np.array(u, np.uint8) for u in units])
        orig = np.repeat(np.arange(len(units)), lens)
        new_id = np.where(gone, -1, np.cumsum(~gone) - 1)
        self.unit_id = new_id[orig].astype(np.int32)
        live = self.unit_id >= 0
        self.pos = np.where(live, np.cumsum(live) - 1, -1).astype(np.int32)
        self.orig = orig
        self.n_units = int((~gone).sum())
        self.len = lens[~gone].astype(np.int32)
        self.first = (np.cumsum(lens) - lens)[~gone].astype(np.int32)
        self.sys = np.array([u[0] == SYS for u, g in zip(units, gone) if not g])
        self.live = int(live.sum())


def _chunk_tags(n):
    video = n - min(25, n // 2)
    mod = np.full(n, VIDEO, np.uint8)
    mod[video:] = AUDIO
    unit = np.zeros(n, np.int32)
    unit[video:] = 1
    return mod, unit


def _plan_keep(c, lay):
    """A plan as the selection leaves it: the system prefix, the newest units and a scattering
    of older ones, within the budget."""
    rng = random.Random(c["slots"] + c["budget"])
    keep = lay.sys.copy()
    left = c["budget"] - int(lay.len[keep].sum())
    order = list(range(lay.n_units - 1, -1, -1))
    head = [u for u in order if not keep[u]][:max(1, lay.n_units // 20)]
    tail = [u for u in order if not keep[u] and u not in set(head)]
    rng.shuffle(tail)
    for u in head + tail:
        if lay.len[u] <= left:
            keep[u] = True
            left -= int(lay.len[u])
    return keep


def _native_pool(c, lay, keep, n_new):
    """Positions of a native pool's slots: the kept units' slots in order, then n_new tokens in
    the lowest run of empty slots.  (key_pos, span, kept, slot of the first new token)."""
    kept_slot = np.zeros(c["slots"], bool)
    ok = lay.unit_id >= 0
    kept_slot[ok] = keep[lay.unit_id[ok]]
    pos = np.where(kept_slot, np.cumsum(kept_slot) - 1, -1).astype(np.int32)
    kept = int(kept_slot.sum())
    pos = np.concatenate([pos, np.full(n_new, -1, np.int32)])
    run, at = 0, 0
    for s in range(len(pos)):
        run = run + 1 if pos[s] < 0 else 0
        if run == n_new:
            at = s - n_new + 1
            break
    pos[at:at + n_new] = kept + np.arange(n_new)
    return pos, int(np.nonzero(pos >= 0)[0][-1]) + 1, kept, at


# -------------------------------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, dtype, unit=None):
    """N(0, 1) values, with an offset N(0, 0.25) per unit (rows of one unit resemble each
    other), drawn layer by layer."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    for layer in out:
        x = torch.randn(shape[1:], generator=g, device="cuda")
        if unit is not None:
            off = 0.5 * torch.randn(int(unit.max()) + 1, generator=g, device="cuda")
            x += off[unit][:, None, None]
        layer.copy_(x)
    return out


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _i32(n):
    return torch.zeros(n, dtype=torch.int32, device="cuda")


def _u8(n):
    return torch.zeros(max(1, n), dtype=torch.uint8, device="cuda")


def _rep(a, layers):
    return _dev(np.tile(a, layers))


def _recent(c):
    return min(c["chunk"], c["budget"])


def _pool_state(c, seed, grammar=False):
    """History pool, chunk, tags and a StreamStep for them."""
    lay = Layout(c, grammar)
    g = _gen(seed)
    dt = torch.float32 if c["f32"] else torch.bfloat16
    layers, chunk = c["layers"], c["chunk"]
    unit = _dev(lay.orig)
    mod, cunit = _chunk_tags(chunk)
    s = dict(kind=c["kind"], lay=lay)
    s["k"] = _normal(g, (layers, c["slots"], c["hkv"], c["d"]), dt, unit)
    if c["kind"] != "plan":
        s["v"] = _normal(g, (layers, c["slots"], c["hkv"], c["d"]), dt, unit)
        s["kc"] = _normal(g, (layers, chunk, c["hkv"], c["d"]), dt)
        s["vc"] = _normal(g, (layers, chunk, c["hkv"], c["d"]), dt)
    if c["kind"] == "step":
        s["q"] = _normal(g, (layers, chunk, c["hq"], c["d"]), dt)
    s["unit_id"], s["modality"], s["pos"] = (_rep(a, layers) for a in
                                             (lay.unit_id, lay.modality, lay.pos))
    s["cmod"], s["cunit"] = _dev(mod), _dev(cunit)
    s["scale"] = 1.0 / math.sqrt(c["d"])
    s["st"] = StreamStep(n_seg=layers, n_slots=c["slots"], n_units=lay.n_units,
                         n_q_heads=c["hq"], n_kv_heads=c["hkv"], head_dim=c["d"],
                         chunk_len=chunk, budget=c["budget"], recent=_recent(c), page_size=64,
                         weights=WEIGHTS, kv_dtype=dt,
                         cap_dst=(_spans_cap(c, lay) if c["kind"] == "spans" else None))
    return s


def _spans_cap(c, lay):
    return lay.live + c["chunk"]         # the low watermark is a target, not a bound


def _spans_params(c):
    """low and high watermark, recent window, sink lengths, text budget."""
    return c["budget"], c["budget"], _recent(c), max(8, c["frame"] * 2 // 5), 16, 1024


def _span_state(c, seed, n_new):
    """A native pool that already holds its n_new newest tokens, and queries for them."""
    lay = Layout(c)
    keep = np.ones(lay.n_units, bool)
    pos, span, kept, _ = _native_pool(c, lay, keep, n_new)
    g = _gen(seed)
    layers, cap = c["layers"], c["slots"] + n_new
    s = dict(kind=c["kind"], traversal=c["traversal"], scale=1.0 / math.sqrt(c["d"]))
    s["k"] = _normal(g, (layers, cap, c["hkv"], c["d"]), torch.bfloat16)
    s["v"] = _normal(g, (layers, cap, c["hkv"], c["d"]), torch.bfloat16)
    s["q"] = _normal(g, (layers, n_new, c["hq"], c["d"]), torch.bfloat16)
    s["key_pos"] = _rep(pos, layers)
    s["span"] = _i32(layers) + span
    s["qpos0"] = _i32(layers) + kept
    s["out"] = torch.zeros(layers, n_new, c["hq"], c["d"], device="cuda")
    s["status"] = _i32(1)
    size = (ot.omnitide_span_attn_workspace_bytes if c["kind"] == "span_attn"
            else ot.omnitide_decode_span_workspace_bytes)
    s["ws"] = _u8(size(layers, cap, n_new, c["hq"], c["hkv"], c["d"]))
    return s


def _native_state(c, seed):
    """A native pool before a step: tags, K and V, the plan of the step, the chunk.  `tags0`
    (and with packing the rows) are the pool as the step finds it, so that a pass can be taken
    again."""
    lay = Layout(c)
    layers, cap, chunk = c["layers"], c["slots"] + c["chunk"], c["chunk"]
    g = _gen(seed)
    keep = _plan_keep(c, lay)
    pad = c["chunk"]
    uid0 = _rep(np.concatenate([lay.unit_id, np.full(pad, -1, np.int32)]), layers)
    pos0 = _rep(np.concatenate([lay.pos, np.full(pad, -1, np.int32)]), layers)
    mod0 = _rep(np.concatenate([lay.modality, np.zeros(pad, np.uint8)]), layers)
    mod, cunit = _chunk_tags(chunk)
    bf = torch.bfloat16
    s = dict(kind="native", lay=lay, pack=c["pack"], traversal=c["traversal"], layers=layers,
             scale=1.0 / math.sqrt(c["d"]), tags0=(uid0, pos0, mod0),
             tags=(uid0.clone(), pos0.clone(), mod0.clone()))
    s["k"] = _normal(g, (layers, cap, c["hkv"], c["d"]), bf)
    s["v"] = _normal(g, (layers, cap, c["hkv"], c["d"]), bf)
    s["kv0"] = (s["k"].clone(), s["v"].clone()) if c["pack"] else None
    s["kc"] = _normal(g, (layers, chunk, c["hkv"], c["d"]), bf)
    s["vc"] = _normal(g, (layers, chunk, c["hkv"], c["d"]), bf)
    s["q"] = _normal(g, (layers, chunk, c["hq"], c["d"]), bf)
    s["keep"], s["unit_len"] = _rep(keep.astype(np.uint8), layers), _rep(lay.len, layers)
    s["cmod"], s["cunit"] = _dev(mod), _dev(cunit)
    s["remap"] = _i32(layers * lay.n_units)
    for name in ("kept", "n_kept", "span", "slot", "cut", "moved"):
        s[name] = _i32(layers)
    s["status"] = _i32(1)
    s["out"] = torch.zeros(layers, chunk, c["hq"], c["d"], device="cuda")
    s["ws_evict"] = _u8(ot.omnitide_evict_native_workspace_bytes(layers, lay.n_units))
    s["ws_place"] = _u8(ot.omnitide_place_chunk_workspace_bytes(layers, cap))
    s["ws_attn"] = _u8(ot.omnitide_span_attn_workspace_bytes(layers, cap, chunk, c["hq"],
                                                             c["hkv"], c["d"]))
    if c["pack"]:
        s["ws_pack"] = _u8(ot.omnitide_pack_suffix_workspace_bytes(ot.BF16, layers, cap,
                                                                   c["hkv"], c["d"]))
    return s


def _rows_state(c, seed):
    """Compacted pools as chunk or decode attention finds them; rows past n_ctx are unused."""
    g = _gen(seed)
    layers, n = c["layers"], c["chunk"] if c["kind"] == "attn" else c["nq"]
    dt = torch.float32 if c.get("f32") else torch.bfloat16
    s = dict(kind=c["kind"], scale=1.0 / math.sqrt(c["d"]))
    s["k"] = _normal(g, (layers, c["cap"], c["hkv"], c["d"]), dt)
    s["v"] = _normal(g, (layers, c["cap"], c["hkv"], c["d"]), dt)
    s["q"] = _normal(g, (layers, n, c["hq"], c["d"]), dt)
    s["n_ctx"] = _dev(np.array(_contexts(c), np.int32))
    out = torch.bfloat16 if c.get("out_bf16") else torch.float32
    s["out"] = torch.zeros(layers, n, c["hq"], c["d"], dtype=out, device="cuda")
    s["status"] = _i32(1)
    if c["kind"] == "attn":
        size = ot.omnitide_attn_workspace_bytes(layers, c["cap"], n, c["hq"], c["hkv"], c["d"],
                                                dtype=ot.F32 if c["f32"] else ot.BF16)
    else:
        size = ot.omnitide_decode_workspace_bytes(layers, c["cap"], n, c["hq"], c["hkv"], c["d"])
    s["ws"] = _u8(size) if size else None
    return s


def _contexts(c):
    """Rows in use per segment: the first `ctx`, streams decoded together up to 10% fewer."""
    rng = random.Random(c["ctx"])
    n = c["chunk"] if c["kind"] == "attn" else c["nq"]
    return [max(n, c["ctx"] - (rng.randint(0, c["ctx"] // 10) if i else 0))
            for i in range(c["layers"])]


def prepare(case, seed):
    c = case
    kind = c["kind"]
    if kind in ("step", "plan"):
        return _pool_state(c, seed)
    if kind == "spans":
        s = _pool_state(c, seed, grammar=True)
        s["params"] = _spans_params(c)
        s["rope"] = ((ROPE_BASE, c["rope"], ot.ROPE_HALF if c["half"] else ot.ROPE_INTERLEAVED)
                     if c["rope"] else None)
        s["st"].score(s["k"], s["unit_id"], s["modality"])
        return s
    if kind == "compact":
        s = _pool_state(c, seed)
        s["keep"] = _rep(_plan_keep(c, s["lay"]).astype(np.uint8), c["layers"])
        s["rope"] = ((ROPE_BASE, c["rope"], ot.ROPE_HALF if c["half"] else ot.ROPE_INTERLEAVED)
                     if c["rope"] else None)
        s["st"].score(s["k"], s["unit_id"], s["modality"])
        return s
    if kind in ("attn", "decode"):
        return _rows_state(c, seed)
    if kind == "native":
        return _native_state(c, seed)
    return _span_state(c, seed, c["chunk"] if kind == "span_attn" else c["nq"])


# ----------------------------------------------------------------------------------- the passes

def _pool_out(st):
    return dict(k=st.k_dst, v=st.v_dst, unit_id=st.unit_id_dst, modality=st.modality_dst,
                pos=st.pos_dst, src=st.src_of_dst, remap=st.unit_remap, n_ctx=st.n_ctx,
                n_pages=st.n_pages, status=st.d_status)


def run(state):
    s, kind = state, state["kind"]
    if kind in ("step", "plan", "spans", "compact"):
        st = s["st"]
        if kind == "step":
            st.run(s["k"], s["v"], s["unit_id"], s["modality"], s["pos"], s["kc"], s["vc"],
                   s["cmod"], s["cunit"], s["q"], s["scale"])
            return dict(out=st.out, wsum=st.unit_wsum, keep=st.keep, kept=st.kept_tokens,
                        **_pool_out(st))
        if kind == "plan":
            st.score(s["k"], s["unit_id"], s["modality"])
            st.select()
            return dict(wsum=st.unit_wsum, len=st.unit_len, first=st.unit_first,
                        last=st.unit_last, flags=st.unit_flags, score=st.unit_score,
                        keep=st.keep, kept=st.kept_tokens, status=st.d_status)
        args = (s["k"], s["v"], s["unit_id"], s["modality"], s["pos"], s["kc"], s["vc"],
                s["cmod"], s["cunit"])
        if kind == "spans":
            st.plan_spans(s["unit_id"], s["modality"], *s["params"])
            st.compact_spans(*args, rope=s["rope"])
            return dict(keep_len=st.keep_len, keep_slot=st.keep_slot, kept=st.kept_tokens,
                        **_pool_out(st))
        st.compact(*args, keep=s["keep"], rope=s["rope"])
        return _pool_out(st)
    if kind == "attn":
        ot.omnitide_chunk_attn(s["q"], s["k"], s["v"], s["n_ctx"], s["scale"], s["out"], s["ws"],
                               s["status"])
        return dict(out=s["out"], status=s["status"])
    if kind == "decode":
        ot.omnitide_decode_attn(s["q"], s["k"], s["v"], s["n_ctx"], s["scale"], s["out"],
                                s["ws"], s["status"])
        return dict(out=s["out"], status=s["status"])
    if kind == "native":
        return _run_native(s)
    call = ot.omnitide_span_attn if kind == "span_attn" else ot.omnitide_decode_span_attn
    call(s["q"], s["k"], s["v"], s["key_pos"], s["span"], s["qpos0"], s["scale"], s["out"],
         s["ws"], s["status"], skip_empty_tiles=s["traversal"] != 0,
         position_order=s["traversal"] == 2)
    return dict(out=s["out"], status=s["status"])


def _run_native(s):
    uid, pos, mod = s["tags"]
    for t, t0 in zip(s["tags"], s["tags0"]):          # the pool as the step finds it
        t.copy_(t0)
    if s["kv0"] is not None:
        s["k"].copy_(s["kv0"][0])
        s["v"].copy_(s["kv0"][1])
    n = s["layers"]
    ot.omnitide_evict_native(uid, pos, n, s["lay"].n_units, s["unit_len"], s["remap"], s["kept"],
                             s["n_kept"], s["span"], s["ws_evict"], keep=s["keep"],
                             d_status=s["status"])
    if s["pack"]:
        ot.omnitide_pack_suffix(s["k"], s["v"], 64, s["pack"], uid, mod, pos, s["span"],
                                s["cut"], s["moved"], s["ws_pack"])
    ot.omnitide_place_chunk(s["k"], s["v"], uid, mod, pos, s["kc"], s["vc"], s["cmod"],
                            s["cunit"], s["kept"], s["n_kept"], s["slot"], s["span"],
                            s["ws_place"], d_status=s["status"])
    ot.omnitide_span_attn(s["q"], s["k"], s["v"], pos, s["span"], s["kept"], s["scale"],
                          s["out"], s["ws_attn"], s["status"],
                          skip_empty_tiles=s["traversal"] != 0,
                          position_order=s["traversal"] == 2)
    return dict(out=s["out"], k=s["k"], v=s["v"], unit_id=uid, pos=pos, modality=mod,
                span=s["span"], kept=s["kept"], n_kept=s["n_kept"], slot=s["slot"],
                cut=s["cut"], moved=s["moved"], remap=s["remap"], status=s["status"])


# ----------------------------------------------------------------------------------------- work

def _attn_work(n_q, ctx, hq, hkv, d, eb, ob):
    """One layer: every query of n_q against its visible keys."""
    pairs = n_q * (ctx - n_q) + n_q * (n_q + 1) / 2
    return dict(bytes=2 * ctx * hkv * d * eb + n_q * hq * d * (eb + ob),
                flops=4.0 * hq * d * pairs)


def work(case):
    c, kind = case, case["kind"]
    hq, hkv, d, layers = c["hq"], c["hkv"], c["d"], c["layers"]
    if kind in ("attn", "decode"):
        n = c["chunk"] if kind == "attn" else c["nq"]
        eb, ob = 4 if c.get("f32") else 2, 2 if c.get("out_bf16") else 4
        w = [_attn_work(n, x, hq, hkv, d, eb, ob) for x in _contexts(c)]
        return dict(bytes=sum(x["bytes"] for x in w), flops=sum(x["flops"] for x in w))
    lay = Layout(c, grammar=kind == "spans")
    if kind in ("span_attn", "decode_span"):
        n = c["chunk"] if kind == "span_attn" else c["nq"]
        w = _attn_work(n, lay.live + n, hq, hkv, d, 2, 4)
        return dict(bytes=layers * (w["bytes"] + 4 * (c["slots"] + n)),
                    flops=layers * w["flops"])
    eb = 4 if c.get("f32") else 2
    row = hkv * d * eb
    score = lay.live * row + 5 * c["slots"] + 24 * lay.n_units
    if kind == "plan":
        return dict(bytes=layers * (score + 33 * lay.n_units), flops=0)
    chunk = c["chunk"]
    if kind == "native":
        kept = int(lay.len[_plan_keep(c, lay)].sum())
        w = _attn_work(chunk, kept + chunk, hq, hkv, d, 2, 4)
        return dict(bytes=layers * (w["bytes"] + 4 * chunk * row + 16 * c["slots"]),
                    flops=layers * w["flops"])
    # kept history: taken as the budget; whole units leave a few percent of it unused (the span
    # plan's low watermark is a target)
    kept = min(c["budget"], lay.live)
    copy = 4 * (kept + chunk) * row + 26 * (kept + chunk) + 13 * lay.n_units
    if kind == "step":
        w = _attn_work(chunk, kept + chunk, hq, hkv, d, eb, 4)
        return dict(bytes=layers * (score + 33 * lay.n_units + copy + w["bytes"]),
                    flops=layers * w["flops"])
    if kind == "spans":
        copy += 6 * c["slots"]
    return dict(bytes=layers * copy, flops=0)


def tolerance(case):
    """Whole numbers are exact.  Chunk attention feeds bf16 probabilities to the products (2^-9
    relative each, against references that another split or tile order places elsewhere): 1.6e-3
    to 2e-3 against 64 bits, 4 times that here.  Decode carries 16 bits of each probability
    (2e-6 to 3e-6 against 64 bits).  A rotated key may round the other way (one bf16 step of a few
    elements, 2^-21 of the pair in float32)."""
    kind = case["kind"]
    if kind == "plan":
        return "exact"
    if kind == "step":                        # values with a unit offset: 1.4e-4 to 9e-4
        return {"rel": 4e-3}
    if kind in ("attn", "span_attn", "native"):
        return {"rel": 8e-3}
    if kind in ("decode", "decode_span"):
        return {"rel": 2e-5}
    if not case["rope"]:
        return "exact"
    return {"rel": 1e-6, "max": 1e-5} if case["f32"] else {"rel": 1e-4, "max": 8e-3}


# ----------------------------------------------------------------------------- 64-bit references

def _attend64(q, k, v, scale, n=None):
    """q [L, hq, d] over rows k, v [n, hkv, d] (the last L are the queries' own), float64."""
    L, hq, d = q.shape
    n, hkv = k.shape[:2]
    out = torch.empty(L, hq, d, dtype=torch.float64, device=q.device)
    hide = (torch.arange(n, device=q.device)[None, :] >
            (n - L + torch.arange(L, device=q.device))[:, None])
    for h in range(hq):
        g = h // (hq // hkv)
        s = (q[:, h].double() @ k[:, g].double().t()) * scale
        s.masked_fill_(hide, -math.inf)
        out[:, h] = torch.softmax(s, -1) @ v[:, g].double()
    return out


def _score64(k, lay):
    """Per-unit weighted key magnitudes of one layer, whole numbers."""
    live = torch.from_numpy(lay.unit_id >= 0).cuda()
    x = (k.double().abs().clamp_(max=32.0) * 65536.0).floor_().sum((1, 2)).long()
    w = torch.tensor([int(round(256 * v)) for v in WEIGHTS] + [int(256 * WEIGHTS[TEXT])])
    x = x * w[torch.from_numpy(lay.modality).long()].cuda()
    out = torch.zeros(lay.n_units, dtype=torch.int64, device="cuda")
    return out.index_add_(0, torch.from_numpy(lay.unit_id).cuda()[live].long(), x[live])


def _select64(c, lay, wsum):
    """Kept units: system units, the newest that fit the window, then by score and id."""
    length = lay.len.astype(np.int64)
    keep = lay.sys.copy()
    left = c["budget"] - int(length[keep].sum())
    window = min(_recent(c), left)
    used = 0
    for u in range(lay.n_units - 1, -1, -1):
        if lay.sys[u]:
            continue
        if used + length[u] > window:
            break
        keep[u] = True
        used += int(length[u])
    left -= used
    score = wsum // length
    rest = [u for u in range(lay.n_units) if not keep[u]]
    for u in sorted(rest, key=lambda i: (-int(score[i]), -i)):
        if length[u] > left:
            break
        keep[u] = True
        left -= int(length[u])
    return keep


def _spans64(c, lay):
    """Per-slot mask of the span plan."""
    low, high, recent, sink_v, sink_a, text_budget = _spans_params(c)
    slots = [np.arange(f, f + n) for f, n in zip(lay.first, lay.len)]
    mask = np.zeros(c["slots"], bool)
    if lay.live <= high:
        mask[lay.unit_id >= 0] = True
        return mask
    newest, used = set(), 0
    for u in range(lay.n_units - 1, -1, -1):
        if lay.sys[u]:
            continue
        if used + lay.len[u] > recent:
            break
        newest.add(u)
        used += int(lay.len[u])
    kept, text_seen = [], 0
    for u in range(lay.n_units):
        m = lay.modality[slots[u]]
        if lay.sys[u] or u in newest:
            kept.append(np.ones(len(m), bool))
            continue
        start = np.concatenate([[True], m[1:] != m[:-1]])
        at = np.arange(len(m))
        place = at - np.maximum.accumulate(np.where(start, at, 0))
        text = m == TEXT
        rank = np.cumsum(text) - 1
        kept.append((m == MARK) | ((m == VIDEO) & (place < sink_v)) |
                    ((m == AUDIO) & (place < sink_a)) | (text & (rank < text_budget - text_seen)))
        text_seen += int(text.sum())
    count = np.array([int(k.sum()) for k in kept])
    order = [u for u in range(lay.n_units) if 0 < count[u] < lay.len[u]]
    order += [u for u in range(lay.n_units) if count[u] == lay.len[u] and not lay.sys[u]]
    for u in order:
        if count.sum() <= low or (count > 0).sum() <= 1:
            break
        count[u] = 0
    for u in range(lay.n_units):
        if count[u]:
            mask[slots[u][kept[u]]] = True
    return mask


def _moved_keys64(c, lay, s, mask):
    """The compacted pools' keys: kept slots in order, turned by their position's change, then
    the chunk; zeros past them."""
    idx = np.nonzero(mask)[0]
    shift = torch.from_numpy(np.arange(len(idx)) - lay.pos[idx]).cuda().double()
    rows = torch.from_numpy(idx).cuda()
    out = torch.zeros(s["st"].k_dst.shape, dtype=torch.float64, device="cuda")
    r = c["rope"]
    theta = ROPE_BASE ** (-2.0 * torch.arange(r // 2, device="cuda", dtype=torch.float64) / r)
    ang = shift[:, None] * theta[None, :]
    cos, sin = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    for i in range(c["layers"]):
        x = s["k"][i][rows].double()
        a, b = (x[..., :r // 2], x[..., r // 2:r]) if c["half"] else (x[..., 0:r:2],
                                                                     x[..., 1:r:2])
        ta, tb = a * cos - b * sin, a * sin + b * cos
        y = x.clone()
        if c["half"]:
            y[..., :r // 2], y[..., r // 2:r] = ta, tb
        else:
            y[..., 0:r:2], y[..., 1:r:2] = ta, tb
        out[i, :len(idx)] = y
        out[i, len(idx):len(idx) + c["chunk"]] = s["kc"][i].double()
    return out


def exact(case, seed):
    """Attention outputs and rotated keys in 64 bits; whole numbers and copied bytes have no
    such value."""
    c, kind = case, case["kind"]
    if kind == "plan" or (kind in ("spans", "compact") and not c["rope"]):
        return None
    s = prepare(c, seed)
    bf = torch.bfloat16
    if kind in ("spans", "compact"):
        lay = s["lay"]
        if kind == "spans":
            mask = _spans64(c, lay)
        else:
            keep = _plan_keep(c, lay)
            mask = (lay.unit_id >= 0) & keep[np.maximum(lay.unit_id, 0)]
        return dict(k=_moved_keys64(c, lay, s, mask))
    out = torch.empty(s["q"].shape, dtype=torch.float64, device="cuda")
    for i in range(c["layers"]):
        q = s["q"][i]
        if kind == "step":
            lay = s["lay"]
            keep = _select64(c, lay, _score64(s["k"][i], lay).cpu().numpy())
            rows = torch.from_numpy(np.nonzero((lay.unit_id >= 0) &
                                               keep[np.maximum(lay.unit_id, 0)])[0]).cuda()
            k, v = (torch.cat([s[a][i][rows], s[b][i]]) for a, b in (("k", "kc"), ("v", "vc")))
        elif kind == "native":
            lay = s["lay"]
            keep = _plan_keep(c, lay)
            rows = torch.from_numpy(np.nonzero((lay.unit_id >= 0) &
                                               keep[np.maximum(lay.unit_id, 0)])[0]).cuda()
            k, v = (torch.cat([s[a][i][rows], s[b][i]]) for a, b in (("k", "kc"), ("v", "vc")))
        elif kind in ("attn", "decode"):
            n = _contexts(c)[i]
            k, v = s["k"][i][:n], s["v"][i][:n]
        else:
            p = s["key_pos"][:s["k"].shape[1]].long()
            rows = torch.nonzero(p >= 0)[:, 0]
            rows = rows[torch.argsort(p[rows])]
            k, v = s["k"][i][rows], s["v"][i][rows]
        # float32 inputs enter the products as bf16 (as the entry point documents)
        out[i] = _attend64(q.to(bf), k.to(bf), v.to(bf), s["scale"])
    return dict(out=out)

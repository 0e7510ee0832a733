"""The work that users of this library have it do, as cases that can be timed and compared.

A case is a dict of plain values.  Five kinds of work cover the library's path in the order a program meets it:

* ``ingest``   a stream's chunks into the cache (mukv_compress_chunk ... mukv_flush)
* ``session``  the same, then questions against it (retrieve and gather)
* ``question`` questions against a cache that is there (retrieve and gather: frames, super-patches, or all three levels)
* ``stores``   questions against three independently compressed caches (retrieve_units, gather_multi)
* ``decode``   new tokens attend to the retrieved rows in place, one call per layer (mukv_attend)
* ``prefill``  a chunk's tokens attend to the retrieved rows and to themselves, one call per layer
               (mukv_prefill_attend), which also yields the chunk's attention signal

Calls are the eager ones of ``paper_2605_22269_amd.binding``.  Inputs are the synthetic streams of
``paper_2605_22269_amd.synth``, drawn on the GPU.  Tables and kept rows come back as views of the context's own memory.
"""
from __future__ import annotations

import math

import torch

from paper_2605_22269_amd import binding as mk
from paper_2605_22269_amd import synth

# ---- what is listed ---------------------------------------------------------------------------------

_7B = dict(layers=28, q_heads=28, kv_heads=4, dim=128, dtype="bf16")
_72B = dict(layers=80, q_heads=64, kv_heads=8, dim=128, dtype="bf16")
_HOUR = dict(frames=3600, tokens=196, unit_frames=1, seg_frames=32, patches=4, keep=0.125)


def listed():
    return [
        # the smallest end-to-end use: half a minute of a small fp32 model, one question
        dict(name="session_tiny_f32", kind="session", layers=1, q_heads=4, kv_heads=1, dim=64, dtype="f32", frames=32,
             tokens=49, unit_frames=1, seg_frames=8, patches=4, keep=0.25, alpha=0.7, chunk=8, batch=1, overlap=0,
             signal="queries", level="frame", questions=1, q_min=16, q_max=16, k_seg=2, k_fine=4),
        # a live stream: the eight frames that just came out of the prefill, compressed at once
        dict(name="live_chunk_7b", kind="ingest", **_7B, **dict(_HOUR, frames=8), alpha=0.7, chunk=8, batch=1, overlap=0,
             signal="queries"),
        # an hour of video ingested in chunks of eight frames, gathered 64 at a time
        dict(name="stream_hour_7b", kind="ingest", **_7B, **_HOUR, alpha=0.7, chunk=8, batch=64, overlap=1,
             signal="queries"),
        # the deep and wide model: few tokens a frame, 80 layers to copy; 20 minutes at 1 frame/s
        dict(name="stream_20min_72b", kind="ingest", **_72B, frames=1200, tokens=64, unit_frames=1, seg_frames=32, patches=4,
             keep=0.125, alpha=0.7, chunk=8, batch=64, overlap=1, signal="queries"),
        # the attention signal handed over by the prefill, so the queries are not read
        dict(name="stream_signal_given_7b", kind="ingest", **_7B, **dict(_HOUR, frames=1000), alpha=0.7, chunk=8, batch=64,
             overlap=1, signal="given"),
        # the coarsest granularity: segments of 32 frames ranked as one unit, 80 % of their tokens kept
        dict(name="segment_units_7b", kind="ingest", **_7B, frames=40, tokens=196, unit_frames=32, seg_frames=1, patches=32,
             keep=0.8, alpha=0.8, chunk=16, batch=1, overlap=1, signal="given"),
        # one question against an hour of video
        dict(name="question_hour_7b", kind="question", **_7B, **_HOUR, level="frame", questions=1, q_min=32, q_max=32,
             k_seg=8, k_fine=32),
        # 64 users' questions of uneven lengths against it in one call
        dict(name="questions64_hour_7b", kind="question", **_7B, **_HOUR, level="frame", questions=64, q_min=16, q_max=64,
             k_seg=8, k_fine=32),
        # one question against three stores with the paper's k, rho and lambda of each
        dict(name="three_stores_7b", kind="stores", **_7B, steps=900, step_frames=4, tokens=196, patches=4, questions=1,
             q_min=32, q_max=32, k_seg=12, k_frame=32, k_patch=20),
        # one user decodes one token through all layers
        dict(name="decode_1_7b", kind="decode", **_7B, **dict(_HOUR, frames=900), questions=1, new=1, local_min=32,
             local_max=32, k_fine=32),
        # 64 users do, with conversations of different lengths
        dict(name="decode_64_7b", kind="decode", **_7B, **dict(_HOUR, frames=900), questions=64, new=1, local_min=16,
             local_max=64, k_fine=32),
        # the prefill of a chunk of eight frames over 32 retrieved frames through all layers
        dict(name="prefill_chunk_7b", kind="prefill", **_7B, **dict(_HOUR, frames=450), questions=1, new=1568, older=0,
             k_fine=32),
    ]


# ---- more cases of the same ranges ------------------------------------------------------------------


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _model(rng, deep=80):
    hq, hkv = rng.choice([(28, 4), (28, 4), (64, 8), (32, 8), (14, 2), (16, 4)])
    return dict(layers=_log(rng, 4, deep), q_heads=hq, kv_heads=hkv, dim=rng.choice([128, 128, 128, 64]),
                dtype=rng.choice(["bf16", "bf16", "bf16", "bf16", "f32"]))


def _frames(rng, lo, hi):
    return dict(frames=_log(rng, lo, hi), tokens=rng.choice([49, 64, 100, 144, 169, 196, 196, rng.randint(40, 256)]),
                unit_frames=1, seg_frames=rng.choice([8, 16, 32, 30]), patches=rng.choice([1, 4, 4, 7]),
                keep=round(rng.uniform(0.08, 0.5), 3))


def draw(rng):
    kind = rng.choice(["ingest", "ingest", "ingest", "units", "session", "question", "question", "stores", "decode",
                       "decode", "prefill", "prefill"])
    while True:
        c = _draw(rng, kind)
        if work(c)["bytes"] <= 8e9 and work(c)["flops"] <= 1.2e12 and _held(c) <= 24e9:
            return c


def _draw(rng, kind):
    if kind in ("ingest", "session"):
        c = dict(kind=kind, **_model(rng), **_frames(rng, 1, 2000), alpha=round(rng.uniform(0.3, 0.9), 2),
                 signal=rng.choice(["queries", "queries", "given"]))
        c["chunk"] = max(-(-c["frames"] // 300), min(c["frames"], rng.choice([1, 2, 4, 8, 8, 16, 32])))
        c["batch"] = rng.choice([1, 1, 8, 64])
        c["overlap"] = rng.choice([0, 1]) if c["frames"] > c["chunk"] * c["batch"] else 0
        if kind == "session":
            c.update(level="frame", **_asked(rng, 4))
        return c
    if kind == "units":
        m = _model(rng, 32)
        p, f = rng.choice([49, 64, 144, 196]), rng.choice([6, 8, 16, 24, 32])
        units = _log(rng, 1, 40)
        return dict(kind="ingest", **m, frames=units, tokens=p, unit_frames=f, seg_frames=1, patches=f,
                    keep=round(rng.uniform(0.3, 0.85), 3), alpha=0.8, chunk=min(units, rng.choice([1, 4, 16])), batch=1,
                    overlap=rng.choice([0, 1]), signal="given")
    if kind == "question":
        return dict(kind=kind, **_model(rng), **_frames(rng, 40, 3600), level=rng.choice(["frame", "frame", "patch", "union"]),
                    **_asked(rng, 64))
    if kind == "stores":
        return dict(kind=kind, **_model(rng, 28), steps=_log(rng, 60, 900), step_frames=rng.choice([2, 4, 8]),
                    tokens=rng.choice([64, 144, 196]), patches=4, questions=_log(rng, 1, 4), q_min=12, q_max=rng.randint(12, 64),
                    k_seg=rng.randint(2, 12), k_frame=rng.randint(4, 32), k_patch=rng.randint(4, 32))
    if kind == "decode":
        return dict(kind=kind, **_model(rng), **_frames(rng, 64, 900), questions=_log(rng, 1, 64), new=rng.choice([1, 1, 1, 4]),
                    local_min=8, local_max=rng.randint(8, 300), k_fine=rng.randint(4, 48))
    c = dict(kind="prefill", **_model(rng, 28), **_frames(rng, 64, 450), questions=rng.choice([1, 1, 2]),
             new=_log(rng, 32, 4000), older=rng.choice([0, 0, rng.randint(1, 200)]), k_fine=rng.choice([0, 8, 32, rng.randint(1, 48)]))
    if c["dtype"] == "f32" or c["dim"] < 128:   # the shapes without matrix-core kernels: short prefills
        c["new"], c["layers"] = min(c["new"], 600), min(c["layers"], 8)
    return c


def _asked(rng, most):
    lo = rng.randint(8, 32)
    return dict(questions=_log(rng, 1, most), q_min=lo, q_max=rng.randint(lo, 64), k_seg=rng.randint(2, 12),
                k_fine=rng.randint(4, 40))


# ---- preparation --------------------------------------------------------------------------------------


def _shape(c):
    return synth.Workload("case", c["layers"], c["q_heads"], c["kv_heads"], c["dim"], c["dtype"], 0, c["tokens"], 1,
                          spike_prob=0.05)


def _esz(c):
    return 2 if c["dtype"] == "bf16" else 4


def _kappa(keep, tokens):
    return max(1, int(math.floor(keep * tokens + 1e-9)))


def _context(c, chunk, questions, **kw):
    unit = c["tokens"] * c["unit_frames"]
    return mk.MuKV(n_layers=c["layers"], n_q_heads=c["q_heads"], n_kv_heads=c["kv_heads"], head_dim=c["dim"],
                   tokens_per_frame=unit, frames_per_segment=c["seg_frames"],
                   superpatches_per_frame=min(c["patches"], unit), dtype=_shape(c).torch_dtype,
                   keep_ratio=max(c["keep"], 1.0 / unit), max_frames=c["frames"], max_chunk_frames=chunk,
                   max_questions=questions, **kw)


def _questions(c, means, seed):
    """Query tokens [sum of lengths][Hq][D] and offsets [B+1]; each question leans towards four frames of the stream."""
    w, dev = _shape(c), means.device
    g = torch.Generator().manual_seed(seed + 1)
    lens = torch.randint(c["q_min"], c["q_max"] + 1, (c["questions"],), generator=g)
    aim = torch.randint(0, means.shape[0], (c["questions"], 4), generator=g).to(dev)
    toks = [synth.planted_question(w, means[aim[b]], int(n), seed + 2 + b, device=dev) for b, n in enumerate(lens)]
    offs = torch.zeros(c["questions"] + 1, dtype=torch.int32)
    offs[1:] = torch.cumsum(lens, 0)
    return torch.cat(toks).contiguous(), offs.to(dev)


def _frame_means(c, k, n):
    return k[-1].view(c["kv_heads"], n, c["tokens"], c["dim"]).float().mean(2).transpose(0, 1).reshape(n, -1)


def _cache(c, seed, questions):
    """A cache filled from a seeded stream, and the mean key of every frame."""
    ctx = _context(c, min(64, c["frames"]), questions, alpha=0.7)
    stream = synth.SynthStream(_shape(c), seed, device="cuda")
    means, left = [], c["frames"]
    while left:
        n = min(64, left)
        k, v, q = stream.next_chunk(n)
        ctx.compress_chunk(k, v, q)
        means.append(_frame_means(c, k, n))
        left -= n
    ctx.flush()
    return ctx, torch.cat(means)


def _rows(c, g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32).to(_shape(c).torch_dtype)


def prepare(case, seed):
    c = case
    s = dict(case=c)
    if c["kind"] in ("ingest", "session"):
        # the chunks as the prefill left them, and a context with room for the stream
        stream = synth.SynthStream(_shape(c), seed, device="cuda", with_q=c["signal"] == "queries")
        sig = None
        if c["signal"] == "given":
            sig = synth.handed_over_attention(c["frames"], c["tokens"] * c["unit_frames"], seed + 3, tie_fraction=0.0).cuda()
        s["chunks"], means, at = [], [], 0
        while at < c["frames"]:
            n = min(c["chunk"], c["frames"] - at)
            k, v, q = stream.next_chunk(n * c["unit_frames"])
            s["chunks"].append((k, v, q, None if sig is None else sig[at:at + n].contiguous()))
            if c["kind"] == "session":
                means.append(_frame_means(c, k, n))
            at += n
        s["ctx"] = _context(c, c["chunk"], c.get("questions", 1), alpha=c["alpha"], batch_chunks=c["batch"],
                            overlap_copy=c["overlap"])
        s["kept"] = _kept(s["ctx"])
        if c["kind"] == "session":
            s["q"], s["offs"] = _questions(c, torch.cat(means), seed)
        return s
    if c["kind"] == "stores":
        return _three_stores(c, seed)
    s["ctx"], means = _cache(c, seed, c["questions"])
    B, L, Hq, Hkv, D = c["questions"], c["layers"], c["q_heads"], c["kv_heads"], c["dim"]
    if c["kind"] == "question":
        s["q"], s["offs"] = _questions(c, means, seed)
        return s
    # decode and prefill: the frames each question retrieved, its own rows of every layer
    host = torch.Generator().manual_seed(seed + 4)
    g = torch.Generator(device="cuda").manual_seed(seed + 5)
    k = min(c["k_fine"], c["frames"])
    s["idx"] = None
    if k:
        s["idx"] = torch.stack([torch.randperm(c["frames"], generator=host)[:k] for _ in range(B)]).to(torch.int32).cuda()
    if c["kind"] == "decode":
        lens = torch.randint(c["local_min"], c["local_max"] + 1, (B,), generator=host)
    else:
        lens = torch.full((B,), c["older"] + c["new"])
    offs = torch.zeros(B + 1, dtype=torch.int32)
    offs[1:] = torch.cumsum(lens, 0)
    n = int(offs[-1])
    s["offs"] = offs.cuda()
    s["q"] = [_rows(c, g, B, c["new"], Hq, D) for _ in range(L)]
    s["k"] = [_rows(c, g, n, Hkv, D) for _ in range(L)]
    s["v"] = [_rows(c, g, n, Hkv, D) for _ in range(L)]
    s["out"] = torch.empty(L, B, c["new"], Hq, D, dtype=_shape(c).torch_dtype, device="cuda")
    s["outs"] = list(s["out"])
    if c["kind"] == "prefill":
        s["signal"] = torch.empty(L, B, c["new"], dtype=torch.float32, device="cuda")
        s["signals"] = list(s["signal"])
        s["ws"] = torch.empty(mk.mukv_prefill_workspace_size(s["ctx"].h, c["new"], k, B), dtype=torch.uint8, device="cuda")
    return s


def _store_specs(c):
    """(unit tokens, units per step, keep ratio, alpha) of the segment, frame and super-patch stores."""
    P, F, S = c["tokens"], c["step_frames"], c["patches"]
    return [(F * P, 1, 0.8, 0.8), (P, 1, 0.1, 0.7), (P // S, S, 0.1, 0.5)]


def _three_stores(c, seed):
    P, F, T = c["tokens"], c["step_frames"], c["steps"]
    per = 8   # steps a call
    stores, sigs = [], []
    for i, (unit, units, keep, alpha) in enumerate(_store_specs(c)):
        stores.append(mk.MuKV(n_layers=c["layers"], n_q_heads=c["q_heads"], n_kv_heads=c["kv_heads"], head_dim=c["dim"],
                              tokens_per_frame=unit, frames_per_segment=1, superpatches_per_frame=1,
                              dtype=_shape(c).torch_dtype, keep_ratio=max(keep, 1.0 / unit), alpha=alpha,
                              max_frames=T * units, max_chunk_frames=per * units, max_questions=c["questions"]))
        sigs.append(synth.handed_over_attention(T * units, unit, seed + 6 + i, tie_fraction=0.0).cuda())
    stream = synth.SynthStream(_shape(c), seed, device="cuda", with_q=False)
    means = []
    for t in range(0, T, per):
        n = min(per, T - t)
        k, v, _ = stream.next_chunk(n * F)
        mid = [x.view(c["layers"], c["kv_heads"], n, F, P, c["dim"])[:, :, :, F // 2].reshape(
            c["layers"], c["kv_heads"], n * P, c["dim"]) for x in (k, v)]
        stores[0].compress_chunk(k, v, None, att_signal=sigs[0][t:t + n])
        stores[1].compress_chunk(*mid, None, att_signal=sigs[1][t:t + n])
        stores[2].compress_chunk(*mid, None, att_signal=sigs[2][t * c["patches"]:(t + n) * c["patches"]])
        means.append(_frame_means(c, mid[0], n))
    s = dict(case=c, stores=stores, ks=[c["k_seg"], c["k_frame"], c["k_patch"]])
    s["rows"] = sum(k * st.kappa for k, st in zip(s["ks"], stores))
    s["q"], s["offs"] = _questions(c, torch.cat(means), seed)
    return s


# ---- views of the context's memory ----------------------------------------------------------------------


class _Memory:
    """Device memory of a context, for torch.as_tensor, which keeps this object (and so the context) alive."""

    def __init__(self, ctx, ptr, shape, kind):
        self.ctx = ctx
        self.__cuda_array_interface__ = dict(shape=tuple(int(n) for n in shape), typestr=kind, data=(int(ptr), False), version=2)


def _kept(ctx):
    """What the compression leaves: kept rows of all layers, kept positions, block keys and values."""
    t, c = mk.mukv_get_state(ctx.h), ctx.cfg
    view = lambda ptr, kind, *shape: torch.as_tensor(_Memory(ctx, ptr, shape, kind), device="cuda")  # noqa: E731
    n, S = c.max_frames, c.superpatches_per_frame
    segs = -(-n // c.frames_per_segment)
    rows = (c.n_layers, c.n_kv_heads, n * t.kappa, c.head_dim)
    out = dict(kept_idx=view(t.kept_idx, "<i4", n, t.kappa), cnt_patch=view(t.cnt_patch, "<i4", n * S))
    for x in "kv":
        raw = view(getattr(t, "store_" + x), "<i2" if ctx.dtype == torch.bfloat16 else "<f4", *rows)
        out["store_" + x] = raw.view(ctx.dtype)
        out["rep_frame_" + x] = view(getattr(t, "rep_frame_" + x), "<f4", n, t.c_kv)
        out["rep_patch_" + x] = view(getattr(t, "rep_patch_" + x), "<f4", n * S, t.c_kv)
        out["rep_seg_" + x] = view(getattr(t, "rep_seg_" + x), "<f4", segs, t.c_kv)
    return out


# ---- one pass --------------------------------------------------------------------------------------------


def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind in ("ingest", "session"):
        ctx = s["ctx"]
        ctx.reset()
        for k, v, q, sig in s["chunks"]:
            ctx.compress_chunk(k, v, q, att_signal=sig)
        ctx.flush()
        if kind == "session":
            return dict(s["kept"], **_ask(s))
        return s["kept"]
    if kind == "question":
        return _ask(s)
    if kind == "stores":
        a, b, d = s["stores"]
        seg = a.retrieve_units(s["q"], s["offs"], s["ks"][0], want_g=True)
        frm = b.retrieve_units(s["q"], s["offs"], s["ks"][1], 0.3, g_in=seg["g"])
        pat = d.retrieve_units(s["q"], s["offs"], s["ks"][2], 0.3, g_in=seg["g"])
        k, v, n = mk.gather_multi([a, b, d], [seg["idx"], frm["idx"], pat["idx"]], [1, 1, c["patches"]], s["rows"])
        return dict(seg=seg, frame=frm, patch=pat, k=k, v=v, n=n)
    ctx = s["ctx"]
    if kind == "decode":
        for layer in range(c["layers"]):
            ctx.attend(layer, s["q"][layer], s["idx"], s["k"][layer], s["v"][layer], s["offs"], True, out=s["outs"][layer])
        return s["out"]
    for layer in range(c["layers"]):
        ctx.prefill_attend(layer, s["q"][layer], s["idx"], s["k"][layer], s["v"][layer], s["offs"], True, out=s["outs"][layer],
                           signal=s["signals"][layer], workspace=s["ws"])
    return s["out"], s["signal"]


def _ask(s):
    c, ctx = s["case"], s["ctx"]
    if c["level"] == "patch":
        hit = ctx.retrieve_patches(s["q"], s["offs"], k_seg=c["k_seg"], k_patch=c["k_fine"])
        k, v, n = ctx.gather_patches(hit["patch_idx"])
        return dict(hit, k=k, v=v, n=n)
    hit = ctx.retrieve(s["q"], s["offs"], k_seg=c["k_seg"], k_frame=c["k_fine"])
    if c["level"] == "union":
        pat = ctx.retrieve_patches(s["q"], s["offs"], k_seg=c["k_seg"], k_patch=c["k_fine"])
        hit.update(pat)
        k, v, n = ctx.gather_union(hit["seg_idx"], hit["frame_idx"], pat["patch_idx"])
    else:
        k, v, n = ctx.gather_kv(hit["frame_idx"])
    return dict(hit, k=k, v=v, n=n)


# ---- what a pass cannot do without -------------------------------------------------------------------------


def _row(c):
    """Bytes of one token's K and V in one layer."""
    return 2 * c["kv_heads"] * c["dim"] * _esz(c)


def _ingest_work(c):
    unit = c["tokens"] * c["unit_frames"]
    keys = unit * c["kv_heads"] * c["dim"] * _esz(c)
    kept = 2 * _kappa(c["keep"], unit) * c["layers"] * _row(c)
    flops = unit * c["kv_heads"] * 5 * c["dim"] * math.log2(c["dim"])      # the transform of every key
    if c["signal"] == "queries":
        keys += unit * c["q_heads"] * c["dim"] * _esz(c)
        flops += unit * (unit + 1) * c["dim"] * c["q_heads"]                # causal scores inside the frame
    else:
        keys += 4 * unit
    return c["frames"] * (keys + kept), c["frames"] * flops


def _ask_work(c):
    C, B = c["kv_heads"] * c["dim"], c["questions"]
    kappa = _kappa(c["keep"], c["tokens"])
    keys = -(-c["frames"] // c["seg_frames"])
    keys += c["frames"] * {"frame": 1, "patch": c["patches"], "union": 1 + c["patches"]}[c["level"]]
    q_bytes = B * 0.5 * (c["q_min"] + c["q_max"]) * c["q_heads"] * c["dim"] * _esz(c)
    k = min(c["k_fine"], c["frames"])
    # rows written; a union's segments hold most of what its other two levels choose
    rows = {"frame": k * kappa, "patch": k * kappa / c["patches"],
            "union": min(c["k_seg"] * c["seg_frames"], c["frames"]) * kappa}[c["level"]]
    read = min(B * rows, c["frames"] * kappa)
    return keys * C * 4 + q_bytes + (B * rows + read) * c["layers"] * _row(c), 2.0 * keys * C * B


def work(case):
    c = case
    if c["kind"] == "ingest":
        b, f = _ingest_work(c)
    elif c["kind"] == "session":
        (b, f), (b2, f2) = _ingest_work(c), _ask_work(c)
        b, f = b + b2, f + f2
    elif c["kind"] == "question":
        b, f = _ask_work(c)
    elif c["kind"] == "stores":
        B, C = c["questions"], c["kv_heads"] * c["dim"]
        b = B * 0.5 * (c["q_min"] + c["q_max"]) * c["q_heads"] * c["dim"] * _esz(c)
        f = 0.0
        for (unit, units, keep, _), k in zip(_store_specs(c), (c["k_seg"], c["k_frame"], c["k_patch"])):
            kap, n = _kappa(keep, unit), c["steps"] * units
            b += n * C * 4 + (B * k + min(B * k, n)) * kap * c["layers"] * _row(c)
            f += 2.0 * n * C * B
    else:
        B, kap = c["questions"], _kappa(c["keep"], c["tokens"])
        past = min(c["k_fine"], c["frames"]) * kap
        unique = min(B * past, c["frames"] * kap)
        if c["kind"] == "decode":
            loc = 0.5 * (c["local_min"] + c["local_max"])
            seen = c["new"] * (past + loc)
        else:
            loc = c["older"] + c["new"]
            seen = c["new"] * (past + c["older"] + 0.5 * (c["new"] + 1))
        b = (unique + B * loc) * _row(c) + 2 * B * c["new"] * c["q_heads"] * c["dim"] * _esz(c)
        b, f = b * c["layers"], 4.0 * B * seen * c["q_heads"] * c["dim"] * c["layers"]
    return dict(bytes=float(b), flops=float(f))


def _held(c):
    """Bytes of the state that prepare() makes, roughly."""
    if c["kind"] in ("ingest", "session"):
        unit = c["tokens"] * c["unit_frames"]
        return c["frames"] * unit * (c["layers"] * _row(c) * (1 + c["keep"]) + c["q_heads"] * c["dim"] * _esz(c)) + work(c)["bytes"]
    if c["kind"] == "stores":
        return c["steps"] * c["step_frames"] * c["tokens"] * c["layers"] * _row(c) + work(c)["bytes"]
    return c["frames"] * _kappa(c["keep"], c["tokens"]) * c["layers"] * _row(c) + 2 * work(c)["bytes"]


# ---- how far another correct implementation may be off ------------------------------------------------------


def tolerance(case):
    if case["kind"] in ("decode", "prefill"):
        # outputs rounded once to the payload type from fp32 sums.  Against the same attention in fp64 the calls are
        # off by rel 1.7e-3 / max 0.024 (bf16) and rel 3.4e-7 / max 6.6e-6 (fp32); the prefill's signal by rel 1e-7
        if case["dtype"] == "f32":
            return {"rel": 2e-6, "max": 4e-5}
        return {"rel": 7e-3, "max": 1e-1}
    # positions, indices and rows are whole numbers and copies; keys and scores are fp64 sums rounded once to float32
    return {"rel": 3e-7, "max": 3e-6, "differ": 0.0}


# ---- the same numbers in 64 bits ------------------------------------------------------------------------------


def exact(case, seed):
    """The attention calls in fp64.  The others return whole numbers, copied rows, and keys and scores that are fp64 sums
    already; a fully independent evaluation of those is what the repository's oracle and its tests are for."""
    c = case
    if c["kind"] not in ("decode", "prefill") or work(c)["flops"] > 1.3e12:
        return None
    s = prepare(c, seed)
    kept, kap = _kept(s["ctx"]), s["ctx"].kappa
    B, n_q, Hq, Hkv, D = c["questions"], c["new"], c["q_heads"], c["kv_heads"], c["dim"]
    G, offs = Hq // Hkv, s["offs"].tolist()
    out = torch.empty(c["layers"], B, n_q, Hq, D, dtype=torch.float64, device="cuda")
    sig = torch.zeros(c["layers"], B, n_q, dtype=torch.float64, device="cuda")
    for b in range(B):
        rows = torch.empty(0, dtype=torch.int64, device="cuda")
        if s["idx"] is not None:
            rows = (s["idx"][b].long()[:, None] * kap + torch.arange(kap, device="cuda")).reshape(-1)
        n_loc = offs[b + 1] - offs[b]
        sees = torch.arange(n_loc, device="cuda")[None] <= torch.arange(n_q, device="cuda")[:, None] + (n_loc - n_q)
        sees = torch.cat([sees.new_ones(n_q, rows.numel()), sees], 1)
        for layer in range(c["layers"]):
            for h in range(Hq):
                k, v = (torch.cat([kept["store_" + x][layer, h // G, rows], s[x][layer][offs[b]:offs[b + 1], h // G]]).double()
                        for x in "kv")
                p = (s["q"][layer][b, :, h].double() @ k.T / math.sqrt(D)).masked_fill(~sees, -math.inf).softmax(1)
                out[layer, b, :, h] = p @ v
                if c["kind"] == "prefill":
                    sig[layer, b] += p[:, -n_q:].sum(0) / (Hq * n_q)
    return out if c["kind"] == "decode" else (out, sig)

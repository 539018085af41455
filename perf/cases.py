"""The work that a program which uses this package has it do, case by case, through its public entry points.

A case is a dict of plain values.  `prepare` makes what such a program holds before the call (inputs on the GPU, the
normalised anchor, caches, workspaces, output buffers), `run` is one pass over it, `work` counts what that pass cannot
do without.  Five kinds of pass:

  prefill    one prompt batch of one image grid: anchor scores, selection and compact merge (civic_compact_prefill),
             then one transformer layer's attention and KV-cache write - as civic_prefill_attn_kv, or, with rotary
             positions, civic_mrope_table, civic_kv_write_rope and civic_prefill_attn_rope over the cache
  ragged     the same for samples of different grids packed along the token axis
  decode     one generated token's attention over the caches of a batch (one context length, or one per sample)
  aggregate  the soft anchor aggregation in front of the visual encoder, token weights included
  compress   KV compression and the visual attention over the compressed keys (one size, or packed items)

Sizes are those of paper_2605_28115_amd.workloads and bench.py, and generic ones between and around them.
"""
from __future__ import annotations

import dataclasses
import math

import numpy as np
import torch

from paper_2605_28115_amd import binding as bd
from paper_2605_28115_amd import workloads as wl

DTYPES = {"fp32": torch.float32, "bf16": torch.bfloat16}


# ------------------------------------------------------------------------------------------------------ the cases
def _prefill(name, **kw):
    w = wl.WORKLOADS[name]
    case = dict(kind="prefill", batch=w.batch, frames=w.frames, height=w.height, width=w.width, cell=w.cell_h,
                cell_floor=w.cell_floor, frame_floor=w.frame_floor, budget=w.budget, text=w.text_len, images=w.images,
                dim=w.dim, q_heads=w.n_q_heads, kv_heads=w.n_kv_heads, head_dim=w.head_dim, dtype=w.dtype,
                causal=w.causal, rope=False)
    case.update(kw)
    return case


def listed():
    heads = dict(q_heads=32, kv_heads=8, head_dim=128)
    return [
        # the smallest call: a 16 x 16 image with a short question in full precision, where launches are everything
        dict(name="tiny", **_prefill("tiny")),
        # one 32 x 32 image on a small language model: the interactive single-image prompt
        dict(name="2b", **_prefill("2b")),
        # the same prompt checked in full precision (what a numerics comparison of the model runs)
        dict(name="2b-fp32", **_prefill("2b", dtype="fp32")),
        # four two-image prompts on a larger model: the benchmark's default workload
        dict(name="8b", **_prefill("8b")),
        # the same batch as a model with rotary positions runs it: table, rotated cache write, rotated queries
        dict(name="8b-rope", **_prefill("8b", rope=True)),
        # the selection applied to a visual encoder's 64 x 64 patch grid: no text, no mask, heads of 72
        dict(name="vit", **_prefill("vit")),
        # sixteen video frames in one long prompt
        dict(name="video", **_prefill("video")),
        # eight prompts of one to two images of different grids in one batch
        dict(name="ragged", kind="ragged", dim=4096, dtype="bf16",
             samples="1x16x16+32 1x32x32+128 2x32x32+256 1x24x24+64 1x32x32+96 2x24x24+128 1x16x16+16 2x32x32+200", **heads),
        # the next token of a single conversation: a few megabytes of cache, latency
        dict(name="decode-one", kind="decode", batch=1, ctx="469", s_max=512, dtype="bf16", q_heads=16, kv_heads=8, head_dim=128),
        # the next token of a serving batch of 64 conversations, every one at a length of its own
        dict(name="decode-serve", kind="decode", batch=64, ctx="117..3584", s_max=3584, dtype="bf16", **heads),
        # 4096 patch embeddings of two images to 1365 anchors, ahead of the visual encoder
        dict(name="aggregate", kind="aggregate", batch=2, tokens=4096, anchors=1365, dim=1152, inv_tau=14.0),
        # the encoder's attention over 256 compressed keys for eight images of different size
        dict(name="compress", kind="compress", rows="1365 341 85 1024 600 341 1365 85", packed=True, memory=256, heads=16, head_dim=72),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _heads(rng):
    q, kv = rng.choice([(4, 2), (8, 8), (16, 8), (16, 16), (16, 4), (32, 8), (32, 4), (28, 4)])
    return dict(q_heads=q, kv_heads=kv, head_dim=rng.choice([64, 64, 72, 96, 128, 128, 128]))


def _samples(text):
    """'2x32x32+200 ...' -> [(frames, height, width, text tokens), ...]"""
    out = []
    for part in text.split():
        grid, t = part.split("+")
        out.append(tuple(int(x) for x in grid.split("x")) + (int(t),))
    return out


def draw(rng):
    """One more case of the ranges above."""
    kind = rng.choice(["prefill", "prefill", "prefill", "ragged", "decode", "decode", "aggregate", "compress"])
    while True:
        if kind == "prefill":
            dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"])
            frames = rng.choice([1, 1, 1, 2, 2, 4, _log(rng, 5, 16)])
            images = frames if frames > 1 and frames <= 4 and rng.random() < 0.5 else 1
            height, width = _log(rng, 8, 64), _log(rng, 8, 64)
            nv = frames * height * width
            h = _heads(rng)
            if dtype == "fp32":
                h["head_dim"] = rng.choice([64, 96, 128])
            rope = h["head_dim"] != 72 and rng.random() < 0.4
            c = dict(kind="prefill", batch=_log(rng, 1, 8), frames=frames, height=height, width=width, cell=rng.choice([2, 4, 4, 8]),
                     cell_floor=rng.choice([0, 1, 1, 2]), frame_floor=rng.choice([0, 0, 16]), budget=nv // rng.choice([2, 3, 3, 4, 8]),
                     text=_log(rng, 8, 640), images=images, dim=rng.choice([256, 1024, 1152, 1536, 2048, 2560, 3584, 4096]),
                     dtype=dtype, causal=rng.random() < 0.85, rope=rope, **h)
        elif kind == "ragged":
            parts = []
            for _ in range(_log(rng, 2, 40)):
                f = rng.choice([1, 1, 1, 2, 3])
                parts.append("%dx%dx%d+%d" % (f, _log(rng, 8, 48), _log(rng, 8, 48), _log(rng, 4, 400)))
            c = dict(kind="ragged", dim=rng.choice([1024, 2048, 3584, 4096]), dtype="bf16", samples=" ".join(parts), **_heads(rng))
        elif kind == "decode":
            batch, top = _log(rng, 1, 96), _log(rng, 64, 4096)
            ctx = "%d" % top if rng.random() < 0.5 else "%d..%d" % (max(1, top // rng.choice([2, 8, 30])), top)
            c = dict(kind="decode", batch=batch, ctx=ctx, s_max=top + _log(rng, 1, 512), dtype=rng.choice(["bf16", "bf16", "bf16", "fp32"]), **_heads(rng))
        elif kind == "aggregate":
            tokens = _log(rng, 256, 4096)
            c = dict(kind="aggregate", batch=_log(rng, 1, 4), tokens=tokens, anchors=max(16, tokens // rng.choice([2, 3, 3, 4, 9])),
                     dim=rng.choice([768, 1024, 1152, 1152, 1280]), inv_tau=float(round(math.exp(rng.uniform(math.log(4.0), math.log(100.0))), 2)))
        else:
            heads, head_dim = rng.choice([(12, 64), (16, 64), (16, 72), (16, 80)])
            if rng.random() < 0.5:
                rows, packed = " ".join(str(_log(rng, 24, 1600)) for _ in range(_log(rng, 2, 24))), True
            else:
                rows, packed = " ".join([str(_log(rng, 64, 2048))] * _log(rng, 1, 8)), False
            c = dict(kind="compress", rows=rows, packed=packed, memory=rng.choice([64, 128, 256, 256, 512]), heads=heads, head_dim=head_dim)
        w = work(c)
        # no dearer than the listed ones: the video prompt in bf16, the small prompt in full precision, the serving batch
        fp32 = c.get("dtype") == "fp32" and c["kind"] != "decode"
        if w["flops"] <= (1.0e9 if fp32 else 9.0e10) and w["bytes"] <= (6.0e7 if fp32 else 5.0e8):
            return c


# ------------------------------------------------------------------------------------------------------- geometry
def _grid(frames, height, width, cell, cell_floor, frame_floor, budget):
    return (frames, height, width, cell, cell, cell_floor, frame_floor, budget)


def _workload(c, batch=None):
    """The case's layout as the package's own shape record (frame starts and position ids come from there)."""
    w = wl.Workload("case", 0, c["batch"] if batch is None else batch, c["frames"], c["height"], c["width"], c["cell"], c["cell"],
                    c["cell_floor"], c["frame_floor"], c["budget"], c["text"], c["dim"], c["q_heads"], c["kv_heads"],
                    c["head_dim"], c["dtype"], c["causal"], "normal", c["images"], 0)
    return dataclasses.replace(w, kept=bd.civic_kept_count(w.grid_tuple()))


def _ragged_workloads(c):
    out = []
    for f, h, w, t in _samples(c["samples"]):
        out.append(_workload(dict(c, batch=1, frames=f, height=h, width=w, cell=4, cell_floor=1, frame_floor=0, budget=f * h * w // 3,
                                  text=t, images=1, causal=True)))
    return out


def _contexts(c):
    """Context lengths of a decode batch: one number, or spread evenly over lo..hi in a fixed shuffled order."""
    if ".." not in c["ctx"]:
        return [int(c["ctx"])] * c["batch"], False
    lo, hi = (int(x) for x in c["ctx"].split(".."))
    n = c["batch"]
    at = [hi if n == 1 else lo + (hi - lo) * i // (n - 1) for i in range(n)]
    step = next(s for s in (37, 41, 43, 47) if math.gcd(s, n) == 1)
    return [at[i * step % n] for i in range(n)], True


def work(case):
    c, kind = case, case["kind"]
    if kind in ("prefill", "ragged"):
        ws = [_workload(c)] if kind == "prefill" else _ragged_workloads(c)
        e = 2 if c["dtype"] == "bf16" else 4
        bts, flops = 4 * c["dim"], 0
        for w in ws:
            b, s, sc, n = w.batch, w.seq_len, w.seq_compact, w.n_visual
            qd, kd = w.n_q_heads * w.head_dim, w.n_kv_heads * w.head_dim
            bts += b * ((s + sc) * w.dim * e + 4 * n + 4 * w.kept + 12 * (s + sc) + 4 * sc)      # hidden, scores, kept, ids, source
            bts += b * sc * e * (2 * qd + 4 * kd)                                                  # q, out; k, v read, caches written
            flops += b * (6 * n * w.dim + 4 * qd * (sc * (sc + 1) // 2 if w.causal else sc * sc))
            if c.get("rope"):
                bts += b * sc * w.head_dim * 4                                                    # the table, written
        return {"bytes": bts, "flops": flops}
    if kind == "decode":
        e = 2 if c["dtype"] == "bf16" else 4
        rows = sum(_contexts(c)[0])
        d = c["head_dim"]
        return {"bytes": e * d * (2 * c["kv_heads"] * rows + 2 * c["batch"] * c["q_heads"]), "flops": 4 * c["q_heads"] * d * rows}
    if kind == "aggregate":
        b, t, m, d = c["batch"], c["tokens"], c["anchors"], c["dim"]
        return {"bytes": 2 * d * (b * t + m + b * m) + 4 * b * t, "flops": 4 * b * t * m * d}
    rows = [int(x) for x in c["rows"].split()]
    wd, s, total = c["heads"] * c["head_dim"], c["memory"], sum(rows)
    assign = total if c["packed"] else rows[0]
    return {"bytes": 2 * wd * (4 * total + 2 * len(rows) * s) + 4 * assign * s, "flops": 8 * total * s * wd}


def tolerance(case):
    # fp32: sums of up to 8192 products in another order, and the logits' share of it through the softmax.
    # bf16: weights and outputs rounded to bf16 (2^-9 each) on fp32 sums; indices and copied rows stay what they are.
    if case.get("dtype") == "fp32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}
    return {"rel": 1e-2, "max": 0.2, "differ": 0.0}


# --------------------------------------------------------------------------------------------------- inputs, passes
class _Randn:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(int(seed))

    def __call__(self, *shape, dtype=torch.float32):
        return torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32).to(dtype)


def _anchor(randn, dim):
    return torch.from_numpy(bd.civic_anchor_normalize((randn(dim) + 0.25).cpu().numpy())).cuda()


def prepare(case, seed):
    c, randn = case, _Randn(seed)
    s = {"kind": c["kind"]}
    dt = DTYPES[c.get("dtype", "bf16")]

    def empty(*shape, dtype=dt):
        return torch.empty(shape, dtype=dtype, device="cuda")

    if c["kind"] == "prefill":
        w = _workload(c)
        b, sc, kv = w.batch, w.seq_compact, (w.n_kv_heads, w.head_dim)
        s.update(grid=bd.make_grid(w.grid_tuple()), starts=wl.frame_starts(w), causal=w.causal, rope=c["rope"],
                 hidden=randn(b, w.seq_len, w.dim, dtype=dt), pos=torch.from_numpy(wl.position_ids(w)).cuda(),
                 anchor=_anchor(randn, w.dim), q=randn(b, sc, w.n_q_heads, w.head_dim, dtype=dt), k=randn(b, sc, *kv, dtype=dt),
                 v=randn(b, sc, *kv, dtype=dt), k_cache=empty(b, kv[0], sc, kv[1]), v_cache=empty(b, kv[0], sc, kv[1]),
                 scores=empty(b, w.n_visual, dtype=torch.float32), kept=empty(b, w.kept, dtype=torch.int32),
                 hidden_c=empty(b, sc, w.dim), pos_c=empty(3, b, sc, dtype=torch.int32), src=empty(b, sc, dtype=torch.int32),
                 out=empty(b, sc, w.n_q_heads, w.head_dim))
        if c["rope"]:
            pairs = w.head_dim // 2
            s.update(axis=(np.arange(pairs) % 3).astype(np.int32),
                     freq=(1.0e6 ** (-np.arange(pairs, dtype=np.float64) / pairs)).astype(np.float32),
                     cos_sin=empty(b, sc, pairs, 2, dtype=torch.float32))
    elif c["kind"] == "ragged":
        ws = _ragged_workloads(c)
        s.update(lens=[w.seq_len for w in ws], grids=[bd.make_grid(w.grid_tuple()) for w in ws], starts=[wl.frame_starts(w) for w in ws])
        seq, _, _, comp = bd.civic_ragged_offsets(s["lens"], s["grids"])
        total, rows, longest = int(seq[-1]), int(comp[-1]), int(np.diff(comp).max())
        h, d = (c["q_heads"], c["kv_heads"]), c["head_dim"]
        s.update(comp=comp, hidden=randn(total, c["dim"], dtype=dt), anchor=_anchor(randn, c["dim"]),
                 pos=torch.from_numpy(np.ascontiguousarray(np.concatenate([wl.position_ids(w)[:, 0] for w in ws], axis=1))).cuda(),
                 q=randn(rows, h[0], d, dtype=dt), k=randn(rows, h[1], d, dtype=dt), v=randn(rows, h[1], d, dtype=dt),
                 k_cache=torch.zeros((len(ws), h[1], longest, d), dtype=dt, device="cuda"), out=empty(rows, h[0], d))
        s["v_cache"] = torch.zeros_like(s["k_cache"])
    elif c["kind"] == "decode":
        ctx, ragged = _contexts(c)
        b, d = c["batch"], c["head_dim"]
        s.update(ragged=ragged, ctx=np.asarray(ctx, dtype=np.int32) if ragged else ctx[0], q=randn(b, c["q_heads"], d, dtype=dt),
                 k_cache=randn(b, c["kv_heads"], c["s_max"], d, dtype=dt), v_cache=randn(b, c["kv_heads"], c["s_max"], d, dtype=dt),
                 out=empty(b, c["q_heads"], d))
        if ragged:
            code = bd.CIVIC_BF16 if dt == torch.bfloat16 else bd.CIVIC_F32
            need = int(bd.lib.civic_decode_attn_ragged_workspace_bytes(code, b, s["ctx"].ctypes.data, c["q_heads"], c["kv_heads"], d))
        else:
            need = bd.civic_decode_attn_workspace_bytes(dt, b, c["q_heads"], c["kv_heads"], d, ctx[0])
        s["workspace"] = empty(max(need, 16), dtype=torch.uint8)
    elif c["kind"] == "aggregate":
        b, t, m, d = c["batch"], c["tokens"], c["anchors"], c["dim"]
        s.update(x0=randn(b, t, d, dtype=dt), anchors=randn(m, d, dtype=dt), inv_tau=c["inv_tau"], z0=empty(b, m, d),
                 workspace=empty(int(bd.lib.civic_anchor_aggregate_workspace_bytes(b, t, m, d)), dtype=torch.uint8))
    else:
        rows = [int(x) for x in c["rows"].split()]
        n, h, d, mem = len(rows), c["heads"], c["head_dim"], c["memory"]
        off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
        lead = (int(off[-1]),) if c["packed"] else (n, rows[0])
        s.update(packed=c["packed"], off=off, q=randn(*lead, h, d, dtype=dt), k=randn(*lead, h, d, dtype=dt), v=randn(*lead, h, d, dtype=dt),
                 # assignment weights: non-negative and peaked
                 r=torch.rand((lead[0] if c["packed"] else rows[0], mem), generator=randn.g, device="cuda") ** 4,
                 k_c=empty(n, mem, h, d), v_c=empty(n, mem, h, d), out=empty(*lead, h, d))
        if c["packed"]:
            need = int(bd.lib.civic_kv_compress_ragged_workspace_bytes(n, off.ctypes.data, mem, h * d))
        else:
            need = int(bd.lib.civic_kv_compress_workspace_bytes(n, rows[0], mem, h * d))
        s["workspace"] = empty(max(need, 16), dtype=torch.uint8)
    return s


def run(s):
    if s["kind"] == "prefill":
        bd.civic_compact_prefill(s["hidden"], s["pos"], s["grid"], s["starts"], s["anchor"], 1.0, scores=s["scores"], kept_idx=s["kept"],
                                 hidden_c=s["hidden_c"], pos_c=s["pos_c"], src_idx=s["src"])
        front = [s["scores"], s["kept"], s["hidden_c"], s["pos_c"], s["src"]]
        if not s["rope"]:
            bd.civic_prefill_attn_kv(s["q"], s["k"], s["v"], s["k_cache"], s["v_cache"], 0, s["causal"], out=s["out"])
            return front + [s["out"], s["k_cache"], s["v_cache"]]
        bd.civic_mrope_table(s["pos_c"], s["axis"], s["freq"], cos_sin=s["cos_sin"])
        bd.civic_kv_write_rope(s["k"], s["v"], s["cos_sin"], s["k_cache"], s["v_cache"], 0)
        bd.civic_prefill_attn_rope(s["q"], s["k_cache"].permute(0, 2, 1, 3), s["v_cache"].permute(0, 2, 1, 3), s["cos_sin"], s["causal"], out=s["out"])
        return front + [s["cos_sin"], s["out"], s["k_cache"], s["v_cache"]]
    if s["kind"] == "ragged":
        front = bd.civic_compact_prefill_ragged(s["hidden"], s["pos"], s["lens"], s["grids"], s["starts"], s["anchor"], 1.0)
        bd.civic_prefill_attn_ragged(s["q"], s["k"], s["v"], s["comp"], True, 0.0, s["k_cache"], s["v_cache"], 0, out=s["out"])
        return list(front) + [s["out"], s["k_cache"], s["v_cache"]]
    if s["kind"] == "decode":
        if s["ragged"]:
            return bd.civic_decode_attn_ragged(s["q"], s["k_cache"], s["v_cache"], s["ctx"], out=s["out"], workspace=s["workspace"])
        return bd.civic_decode_attn(s["q"], s["k_cache"], s["v_cache"], s["ctx"], out=s["out"], workspace=s["workspace"])
    if s["kind"] == "aggregate":
        z0, weight = bd.civic_anchor_aggregate(s["x0"], s["anchors"], s["inv_tau"], True, z0=s["z0"], workspace=s["workspace"])
        return [z0, weight]
    if s["packed"]:
        bd.civic_kv_compress_ragged(s["k"], s["v"], s["r"], s["off"], k_c=s["k_c"], v_c=s["v_c"], workspace=s["workspace"])
        bd.civic_cross_attn_ragged(s["q"], s["k_c"], s["v_c"], s["off"], out=s["out"])
    else:
        bd.civic_kv_compress(s["k"], s["v"], s["r"], k_c=s["k_c"], v_c=s["v_c"], workspace=s["workspace"])
        bd.civic_cross_attn(s["q"], s["k_c"], s["v_c"], out=s["out"])
    return [s["k_c"], s["v_c"], s["out"]]

"""CPU-only checks of the C-ABI library: it loads, exports every symbol the header declares, the
host-side functions agree with the tabulated grids, and every documented argument error is
rejected before any HIP call (no compute call is made here)."""
import ctypes as C
import os
import re

import numpy as np
import pytest

from paper_2605_28115_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def bd():
    from paper_2605_28115_amd import binding
    return binding


def test_exports_every_declared_symbol(bd):
    header = open(os.path.join(ROOT, "include", "civic.h")).read()
    declared = set(re.findall(r"\b(civic_[a-z_]+)\s*\(", header))
    assert declared == set(bd.EXPORTS)
    for name in declared:
        assert hasattr(bd.lib, name), name
    assert bd.lib.civic_last_hip_error() == 0


def test_header_limits_match_binding(bd):
    header = open(os.path.join(ROOT, "include", "civic.h")).read()
    lim = dict(re.findall(r"#define (CIVIC_MAX_[A-Z_]+)\s+(\d+)", header))
    assert int(lim["CIVIC_MAX_VISUAL_TOKENS"]) == bd.MAX_VISUAL_TOKENS
    assert int(lim["CIVIC_MAX_FRAMES"]) == bd.MAX_FRAMES
    assert int(lim["CIVIC_MAX_SCORE_DIM"]) == bd.MAX_SCORE_DIM
    assert int(lim["CIVIC_MAX_HEAD_DIM"]) == bd.MAX_HEAD_DIM


@pytest.mark.parametrize("name", list(wl.WORKLOADS))
def test_kept_count_of_tabulated_workloads(bd, name):
    w = wl.WORKLOADS[name]
    assert bd.civic_kept_count(w.grid_tuple()) == w.kept
    assert bd.civic_select_workspace_bytes(w.grid_tuple(), w.batch) == 0
    assert bd.civic_compact_workspace_bytes(w.batch, w.seq_len) == 0


def test_kept_count_closed_form_on_ragged_grids(bd):
    for grid in wl.small_grid_cases():
        frames, H, W, ch, cw, cf, ff, budget = grid
        per_frame = 0
        for r0 in range(0, H, ch):
            for c0 in range(0, W, cw):
                per_frame += min(cf, (min(r0 + ch, H) - r0) * (min(c0 + cw, W) - c0))
        per_frame += min(ff, H * W - per_frame)
        assert bd.civic_kept_count(grid) == max(budget, frames * per_frame), grid


@pytest.mark.parametrize("grid", [
    (0, 4, 4, 2, 2, 1, 0, 1), (1, 0, 4, 2, 2, 1, 0, 1), (1, 4, -1, 2, 2, 1, 0, 1), (1, 4, 4, 0, 2, 1, 0, 1),
    (1, 4, 4, 2, 0, 1, 0, 1), (1, 4, 4, 2, 2, -1, 0, 1), (1, 4, 4, 2, 2, 1, -1, 1), (1, 4, 4, 2, 2, 1, 0, -1),
    (1, 4, 4, 2, 2, 1, 0, 17), (70000, 70000, 2, 2, 2, 1, 0, 1),
])
def test_bad_grids_are_rejected(bd, grid):
    assert bd.lib.civic_kept_count(C.byref(bd.make_grid(grid))) == bd.ERR_INVALID_ARG
    assert bd.lib.civic_kept_count(None) == bd.ERR_INVALID_ARG
    fake = C.c_void_p(0x1000)
    assert bd.lib.civic_select(fake, 1, C.byref(bd.make_grid(grid)), fake, None, None, 0, None) == bd.ERR_INVALID_ARG


def test_anchor_normalize_host(bd):
    rng = np.random.default_rng(0)
    a = (rng.standard_normal(300) * 2 + 5).astype(np.float32)
    q = bd.civic_anchor_normalize(a)
    assert abs(float(q.astype(np.float64).sum())) < 1e-5 and abs(float((q.astype(np.float64) ** 2).sum()) - 1) < 1e-6
    c = a.astype(np.float64) - a.astype(np.float64).mean()
    assert np.abs(q - c / np.linalg.norm(c)).max() < 1e-7
    with pytest.raises(bd.CivicError):
        bd.civic_anchor_normalize(np.full(8, 3.0, dtype=np.float32))
    assert bd.lib.civic_anchor_normalize(None, 8, None) == bd.ERR_INVALID_ARG


def test_argument_errors_precede_any_hip_call(bd):
    L, F, I = bd.lib, C.c_void_p(0x1000), bd.ERR_INVALID_ARG
    odd = C.c_void_p(0x1004)
    st = (C.c_int64 * 3)(1024, 128, 128)
    g = bd.make_grid((1, 4, 4, 2, 2, 1, 0, 5))
    # civic_score: null, bad dtype, dim not a vector multiple, stride < dim, misaligned, too wide
    assert L.civic_score(None, 1, 4, 64, 64, F, 1.0, F, None) == I
    assert L.civic_score(F, 7, 4, 64, 64, F, 1.0, F, None) == I
    assert L.civic_score(F, 1, 4, 64, 60, F, 1.0, F, None) == I
    assert L.civic_score(F, 1, 4, 32, 64, F, 1.0, F, None) == I
    assert L.civic_score(odd, 1, 4, 64, 64, F, 1.0, F, None) == I
    assert L.civic_score(F, 1, -1, 64, 64, F, 1.0, F, None) == I
    assert L.civic_score(F, 1, 4, 16384, 16384, F, 1.0, F, None) == bd.ERR_UNSUPPORTED
    assert L.civic_score(F, 1, 0, 64, 64, F, 1.0, F, None) == bd.CIVIC_OK          # nothing to do
    # civic_score_visual: the same checks plus the frame spans
    def score_vis(fs, seq_len=40, grid=g, hidden=F, dim=64, batch=1, dt=1, scores=F, anchor=F):
        arr = np.asarray(fs, dtype=np.int64)
        return L.civic_score_visual(hidden, dt, batch, seq_len, dim, C.byref(grid), C.c_void_p(arr.ctypes.data), anchor,
                                    C.c_float(1.0), scores, None)
    assert score_vis([30]) == I and score_vis([-1]) == I and score_vis([0], seq_len=15) == I
    assert score_vis([0], hidden=None) == I and score_vis([0], hidden=odd) == I and score_vis([0], dim=60) == I
    assert score_vis([0], dt=5) == I and score_vis([0], scores=None) == I and score_vis([0], anchor=None) == I
    assert score_vis([0], batch=-1) == I and score_vis([0], batch=0, hidden=None, scores=None) == bd.CIVIC_OK
    assert score_vis([0], dim=16384) == bd.ERR_UNSUPPORTED and score_vis([0], batch=70000) == bd.ERR_UNSUPPORTED
    two = bd.make_grid((2, 4, 4, 2, 2, 1, 0, 5))
    assert score_vis([0, 8], grid=two) == I and score_vis([20, 0], grid=two) == I
    assert L.civic_score_visual(F, 1, 1, 40, 64, C.byref(g), None, F, C.c_float(1.0), F, None) == I
    # civic_select: null scores / output, too many tokens
    assert L.civic_select(None, 1, C.byref(g), F, None, None, 0, None) == I
    assert L.civic_select(F, 1, C.byref(g), None, None, None, 0, None) == I
    assert L.civic_select(F, -1, C.byref(g), F, None, None, 0, None) == I
    big = bd.make_grid((1, 256, 256, 4, 4, 1, 0, 100))
    assert L.civic_select(F, 1, C.byref(big), F, None, None, 0, None) == bd.ERR_UNSUPPORTED
    assert L.civic_select(F, 0, C.byref(g), F, None, None, 0, None) == bd.CIVIC_OK
    # civic_compact: frame spans out of range / overlapping / not ascending, seq shorter than N_v
    def compact(fs, seq_len=40, n_kept=5, grid=g, hidden=F, dim=64):
        arr = np.asarray(fs, dtype=np.int64)
        return L.civic_compact(hidden, 1, dim, F, 1, seq_len, C.byref(grid), C.c_void_p(arr.ctypes.data), F, n_kept,
                               F, F, F, None, 0, None)
    assert compact([30]) == I and compact([-1]) == I and compact([0], seq_len=15) == I
    assert compact([0], n_kept=17) == I and compact([0], hidden=None) == I and compact([0], hidden=odd) == I
    g2 = bd.make_grid((2, 4, 4, 2, 2, 1, 0, 5))
    assert compact([0, 8], grid=g2) == I and compact([20, 0], grid=g2) == I
    many = bd.make_grid((200, 1, 1, 1, 1, 0, 0, 5))
    assert compact(list(range(200)), seq_len=400, grid=many) == bd.ERR_UNSUPPORTED
    # civic_compact_prefill: the checks of all three stages, before anything is launched
    def front(fs=(0,), seq_len=40, grid=g, hidden=F, dim=64, batch=1, pos=F, anchor=F, scores=F, kept=F, hc=F, pc=F, si=F):
        arr = np.asarray(fs, dtype=np.int64)
        return L.civic_compact_prefill(hidden, 1, batch, seq_len, dim, pos, C.byref(grid), C.c_void_p(arr.ctypes.data), anchor,
                                       C.c_float(1.0), scores, kept, hc, pc, si, None, 0, None)
    assert front(fs=[30]) == I and front(seq_len=15) == I and front(hidden=None) == I and front(hidden=odd) == I
    assert front(dim=60) == I and front(anchor=None) == I and front(scores=None) == I and front(kept=None) == I
    assert front(pos=None) == I and front(hc=None) == I and front(pc=None) == I and front(si=None) == I
    assert front(kept=C.c_void_p(0x1002)) == I and front(batch=-1) == I
    assert front(grid=big, seq_len=70000) == bd.ERR_UNSUPPORTED and front(dim=16384) == bd.ERR_UNSUPPORTED
    assert front(batch=0, hidden=None, pos=None, scores=None, kept=None, hc=None, pc=None, si=None) == bd.CIVIC_OK
    # civic_prefill_attn: head mismatch, head_dim, alignment, scale
    def attn(**kw):
        a = dict(q=F, k=F, v=F, o=F, dt=1, b=1, s=8, hq=4, hkv=2, d=64, qs=st, ks=st, os=st, causal=1, scale=0.0)
        a.update(kw)
        return L.civic_prefill_attn(a["q"], a["k"], a["v"], a["o"], a["dt"], a["b"], a["s"], a["hq"], a["hkv"], a["d"],
                                    a["qs"], a["ks"], a["os"], a["causal"], C.c_float(a["scale"]), None)
    assert attn(hq=3) == I and attn(d=60) == I and attn(q=odd) == I and attn(k=None) == I and attn(dt=2) == I
    assert attn(scale=-1.0) == I and attn(scale=float("nan")) == I and attn(qs=None) == I
    assert attn(qs=(C.c_int64 * 3)(1024, 100, 68)) == I
    assert attn(d=512) == bd.ERR_UNSUPPORTED and attn(s=0) == bd.CIVIC_OK
    # civic_kv_write: rows past the cache end, negative pos0, head bytes not a vector multiple
    def kvw(**kw):
        a = dict(k=F, v=F, st=st, dt=1, kc=F, vc=F, b=1, s=8, h=2, d=64, smax=16, pos0=0)
        a.update(kw)
        return L.civic_kv_write(a["k"], a["v"], a["st"], a["dt"], a["kc"], a["vc"], a["b"], a["s"], a["h"], a["d"],
                                a["smax"], a["pos0"], None)
    assert kvw(pos0=9) == I and kvw(pos0=-1) == I and kvw(d=4) == I and kvw(kc=None) == I and kvw(v=odd) == I
    assert kvw(st=None) == I and kvw(h=0) == I and kvw(s=0) == bd.CIVIC_OK
    # civic_prefill_attn_kv: the checks of both calls, and the caches are mandatory
    def attn_kv(**kw):
        a = dict(q=F, k=F, v=F, o=F, kc=F, vc=F, dt=1, b=1, s=8, hq=4, hkv=2, d=64, qs=st, ks=st, os=st, smax=16, pos0=0,
                 causal=1, scale=0.0)
        a.update(kw)
        return L.civic_prefill_attn_kv(a["q"], a["k"], a["v"], a["o"], a["kc"], a["vc"], a["dt"], a["b"], a["s"], a["hq"],
                                       a["hkv"], a["d"], a["qs"], a["ks"], a["os"], a["smax"], a["pos0"], a["causal"],
                                       C.c_float(a["scale"]), None)
    assert attn_kv(kc=None) == I and attn_kv(vc=None) == I and attn_kv(vc=odd) == I
    assert attn_kv(pos0=9) == I and attn_kv(pos0=-1) == I and attn_kv(smax=7) == I
    assert attn_kv(hq=3) == I and attn_kv(d=60) == I and attn_kv(scale=-1.0) == I and attn_kv(ks=None) == I
    # civic_decode_attn: context outside the cache, empty context, head mismatch, alignment, workspace
    def dec(**kw):
        a = dict(q=F, kc=F, vc=F, o=F, dt=1, b=2, hq=4, hkv=2, d=64, smax=100, n=50, scale=0.0, ws=F, wsb=1 << 30)
        a.update(kw)
        return L.civic_decode_attn(a["q"], a["kc"], a["vc"], a["o"], a["dt"], a["b"], a["hq"], a["hkv"], a["d"], a["smax"],
                                   a["n"], C.c_float(a["scale"]), a["ws"], a["wsb"], None)
    assert dec(n=101) == I and dec(n=0) == I and dec(n=-1) == I and dec(hq=3) == I and dec(d=60) == I
    assert dec(q=None) == I and dec(kc=odd) == I and dec(o=None) == I and dec(dt=3) == I and dec(scale=-1.0) == I
    assert dec(d=1024) == bd.ERR_UNSUPPORTED and dec(b=0, q=None, kc=None, vc=None, o=None) == bd.CIVIC_OK
    need = bd.civic_decode_attn_workspace_bytes(__import__("torch").bfloat16, 2, 4, 2, 64, 50)
    assert need == 0                                        # 50 rows are one round of one workgroup: nothing to combine
    need = bd.civic_decode_attn_workspace_bytes(__import__("torch").bfloat16, 2, 4, 2, 64, 5000)
    assert need > 0 and need % 4 == 0
    assert dec(smax=6000, n=5000, ws=None, wsb=0) == bd.ERR_WORKSPACE
    assert dec(smax=6000, n=5000, wsb=need - 4) == bd.ERR_WORKSPACE and dec(smax=6000, n=5000, ws=odd) == bd.ERR_WORKSPACE
    # rotary calls: tables, head sizes, alignment, cache bounds
    ax = np.asarray([0, 1, 2, 1], dtype=np.int32); fr = np.asarray([1.0, 0.5, 0.25, 0.1], dtype=np.float32)
    def table(axis=ax, freq=fr, n=4, pos=F, out=F, b=1, s=8):
        return L.civic_mrope_table(pos, b, s, n, C.c_void_p(axis.ctypes.data) if axis is not None else None,
                                   C.c_void_p(freq.ctypes.data) if freq is not None else None, out, None)
    assert table(axis=None) == I and table(freq=None) == I and table(n=0) == I and table(pos=None) == I and table(out=odd) == I
    assert table(axis=np.asarray([0, 3, 0, 0], dtype=np.int32)) == I
    assert table(freq=np.asarray([1.0, np.inf, 0.0, 0.0], dtype=np.float32)) == I
    assert table(n=129, axis=np.zeros(129, dtype=np.int32), freq=np.zeros(129, dtype=np.float32)) == bd.ERR_UNSUPPORTED
    assert table(s=0, pos=None, out=None) == bd.CIVIC_OK
    def apply(**kw):
        a = dict(x=F, o=F, dt=1, b=1, s=8, h=2, d=64, xs=st, os=st, cs=F)
        a.update(kw)
        return L.civic_mrope_apply(a["x"], a["o"], a["dt"], a["b"], a["s"], a["h"], a["d"], a["xs"], a["os"], a["cs"], None)
    assert apply(d=24) == I and apply(d=63) == I and apply(x=None) == I and apply(cs=None) == I and apply(o=odd) == I
    assert apply(xs=None) == I and apply(dt=9) == I and apply(d=512) == bd.ERR_UNSUPPORTED and apply(s=0, x=None, o=None, cs=None) == bd.CIVIC_OK
    def kvr(**kw):
        a = dict(k=F, v=F, st=st, dt=1, cs=F, kc=F, vc=F, b=1, s=8, h=2, d=64, smax=16, pos0=0)
        a.update(kw)
        return L.civic_kv_write_rope(a["k"], a["v"], a["st"], a["dt"], a["cs"], a["kc"], a["vc"], a["b"], a["s"], a["h"], a["d"],
                                     a["smax"], a["pos0"], None)
    assert kvr(pos0=9) == I and kvr(d=24) == I and kvr(cs=None) == I and kvr(kc=None) == I and kvr(cs=odd) == I and kvr(s=0) == bd.CIVIC_OK
    def attn_rope(**kw):
        a = dict(q=F, k=F, v=F, o=F, dt=1, b=1, s=8, hq=4, hkv=2, d=64, qs=st, ks=st, os=st, causal=1, scale=0.0, cs=F)
        a.update(kw)
        return L.civic_prefill_attn_rope(a["q"], a["k"], a["v"], a["o"], a["dt"], a["b"], a["s"], a["hq"], a["hkv"], a["d"],
                                         a["qs"], a["ks"], a["os"], a["causal"], C.c_float(a["scale"]), a["cs"], None)
    assert attn_rope(cs=None) == I and attn_rope(cs=odd) == I and attn_rope(hq=3) == I and attn_rope(s=0, cs=None) == bd.CIVIC_OK
    # encoder-side calls
    def agg(**kw):
        a = dict(x=F, a=F, dt=1, b=1, t=100, m=10, d=64, tau=1.0, z=F, tw=None, ws=F, wsb=1 << 40)
        a.update(kw)
        return L.civic_anchor_aggregate(a["x"], a["a"], a["dt"], a["b"], a["t"], a["m"], a["d"], C.c_float(a["tau"]), a["z"], a["tw"],
                                        a["ws"], a["wsb"], None)
    assert agg(x=None) == I and agg(a=odd) == I and agg(t=0) == I and agg(m=0) == I and agg(tau=-1.0) == I and agg(dt=4) == I
    assert agg(d=72) == bd.ERR_UNSUPPORTED and agg(dt=0) == bd.ERR_UNSUPPORTED
    assert agg(ws=None) == bd.ERR_WORKSPACE and agg(wsb=1000) == bd.ERR_WORKSPACE
    assert bd.lib.civic_anchor_aggregate_workspace_bytes(1, 100, 10, 64) > 0 and bd.lib.civic_anchor_aggregate_workspace_bytes(1, 0, 10, 64) == 0
    assert agg(b=0, x=None, z=None) == bd.CIVIC_OK
    def comp(**kw):
        a = dict(k=F, v=F, dt=1, r=F, b=1, m=100, s=10, w=64, kc=F, vc=F, ws=F, wsb=1 << 40)
        a.update(kw)
        return L.civic_kv_compress(a["k"], a["v"], a["dt"], a["r"], a["b"], a["m"], a["s"], a["w"], a["kc"], a["vc"], a["ws"], a["wsb"], None)
    assert comp(k=None) == I and comp(r=None) == I and comp(m=0) == I and comp(s=0) == I and comp(vc=odd) == I
    assert comp(dt=0) == bd.ERR_UNSUPPORTED and comp(ws=None) == bd.ERR_WORKSPACE and comp(wsb=10) == bd.ERR_WORKSPACE
    def cross(**kw):
        a = dict(q=F, k=F, v=F, o=F, dt=1, b=1, nq=8, nkv=5, hq=4, hkv=2, d=64, qs=st, ks=st, os=st, scale=0.0)
        a.update(kw)
        return L.civic_cross_attn(a["q"], a["k"], a["v"], a["o"], a["dt"], a["b"], a["nq"], a["nkv"], a["hq"], a["hkv"], a["d"],
                                  a["qs"], a["ks"], a["os"], C.c_float(a["scale"]), None)
    assert cross(nkv=0) == I and cross(nkv=-1) == I and cross(hq=3) == I and cross(k=None) == I and cross(nq=0, nkv=0) == bd.CIVIC_OK
    # a tensor without elements needs no pointer: NULL is accepted exactly then
    OK = bd.CIVIC_OK
    assert L.civic_score(None, 1, 0, 64, 64, F, 1.0, None, None) == OK and L.civic_score(F, 1, 0, 64, 64, None, 1.0, F, None) == I
    assert L.civic_select(None, 0, C.byref(g), None, None, None, 0, None) == OK
    none_kept = bd.make_grid((1, 4, 4, 2, 2, 0, 0, 0))
    fs0 = np.zeros(1, dtype=np.int64)
    def compact0(batch, seq_len, n_kept, out):
        return L.civic_compact(F if batch else None, 1, 64, F if batch else None, batch, seq_len, C.byref(none_kept),
                               C.c_void_p(fs0.ctypes.data), None, n_kept, out, out, out, None, 0, None)
    assert compact0(0, 16, 0, None) == OK                # empty batch
    assert compact0(1, 16, 0, None) == OK                # no text, nothing kept: S_c = 0
    assert compact0(1, 17, 0, None) == I                 # one text token: outputs are needed
    assert attn(q=None, k=None, v=None, o=None, s=0) == OK and attn(q=None, k=None, v=None, o=None, b=0) == OK
    assert kvw(k=None, v=None, kc=None, vc=None, s=0) == OK and kvw(k=None, v=None, kc=None, vc=None, b=0) == OK
    assert attn_kv(q=None, k=None, v=None, o=None, kc=None, vc=None, s=0) == OK
    wide = (C.c_int64 * 3)(8192, 1024, 512)
    assert attn_kv(d=512, qs=wide, ks=wide, os=wide) == bd.ERR_UNSUPPORTED and attn_kv(s=0) == bd.CIVIC_OK
    # ragged Eq. 9 calls: offsets (null, not starting at 0, an empty item), row alignment, workspace
    def offs(*v):
        return np.asarray(v, dtype=np.int64)
    def rcomp(off=offs(0, 5, 12), batch=2, k=F, r=F, n_mem=8, width=64, ws=F, wsb=1 << 30, dt=1):
        return L.civic_kv_compress_ragged(k, F, dt, r, batch, C.c_void_p(off.ctypes.data) if off is not None else None, n_mem, width,
                                          F, F, ws, wsb, None)
    assert rcomp(off=None) == I and rcomp(off=offs(1, 5, 12)) == I and rcomp(off=offs(0, 5, 5)) == I and rcomp(off=offs(0, 5, 3)) == I
    assert rcomp(k=None) == I and rcomp(r=None) == I and rcomp(k=odd) == I and rcomp(batch=-1) == I and rcomp(dt=9) == I
    assert rcomp(width=60) == bd.ERR_UNSUPPORTED and rcomp(n_mem=6) == bd.ERR_UNSUPPORTED and rcomp(dt=0) == bd.ERR_UNSUPPORTED
    assert rcomp(ws=None, wsb=0) == bd.ERR_WORKSPACE and rcomp(wsb=16) == bd.ERR_WORKSPACE and rcomp(batch=0, off=None) == OK
    o3 = offs(0, 5, 12)
    need = L.civic_kv_compress_ragged_workspace_bytes(2, C.c_void_p(o3.ctypes.data), 8, 64)
    # per item 32 rows of partial column sums and Rbar^T (S x its rows rounded up to 64, bf16)
    a256 = lambda x: (x + 255) // 256 * 256
    assert need == a256(2 * 8 * 4 * 32) + a256(8 * (64 + 64) * 2)
    def rattn(off=offs(0, 5, 12), batch=2, q=F, k=F, o=F, hq=4, hkv=2, d=64, qs=st, ks=st):
        return L.civic_cross_attn_ragged(q, k, k, o, 1, batch, C.c_void_p(off.ctypes.data) if off is not None else None, 8, hq, hkv, d,
                                         qs, ks, st, C.c_float(0.0), None)
    assert rattn(off=None) == I and rattn(off=offs(2, 5, 12)) == I and rattn(off=offs(0, 5, 5)) == I and rattn(q=None) == I
    assert rattn(hq=3) == I and rattn(d=60) == I and rattn(qs=None) == I and rattn(k=odd) == I and rattn(batch=0, off=None) == OK
    assert bd.lib.civic_last_hip_error() == 0


def test_kernel_timer_argument_checks(bd):
    # only the handles' values are looked at here: nothing is launched, so nothing touches them
    one, two = C.c_void_p(0x1000), C.c_void_p(0x2000)
    f = bd.lib.civic_time_next_kernel
    assert f(one, None) == bd.ERR_INVALID_ARG
    assert f(None, two) == bd.ERR_INVALID_ARG
    assert f(one, one) == bd.ERR_INVALID_ARG
    assert f(one, two) == bd.CIVIC_OK
    assert f(None, None) == bd.CIVIC_OK             # disarmed again: no later launch of this thread sees the handles


def test_ragged_path_offsets_and_argument_errors(bd):
    """civic_ragged_offsets is a host function (checked against the oracle's own count); the two ragged path calls
    reject every documented error before any HIP call."""
    import oracle
    L = bd.lib
    I, OK = bd.ERR_INVALID_ARG, bd.CIVIC_OK
    grids = [(1, 16, 16, 4, 4, 2, 0, 85), (2, 5, 7, 2, 3, 1, 2, 20), (1, 1, 1, 1, 1, 0, 0, 0), (16, 24, 24, 4, 4, 1, 16, 3072)]
    lens = [288, 90, 1, 9728]
    got = bd.civic_ragged_offsets(lens, grids)
    ref = oracle.ragged_offsets(lens, grids)
    for a, b in zip(got, ref):
        assert np.array_equal(a, b)
    gs = (bd.Grid * 2)(bd.make_grid(grids[0]), bd.make_grid(grids[1]))
    off = lambda *v: np.asarray(v, dtype=np.int64)
    out = np.zeros(3, dtype=np.int64)
    P = lambda a: C.c_void_p(a.ctypes.data) if a is not None else None
    ro = lambda o=off(0, 288, 378), g=gs, b=2: L.civic_ragged_offsets(b, P(o), g, P(out), None, None)
    assert ro() == OK and out.tolist() == [0, 256, 326]
    assert ro(o=None) == I and ro(o=off(1, 288, 378)) == I and ro(o=off(0, 255, 378)) == I and ro(g=None) == I and ro(b=-1) == I
    bad = (bd.Grid * 2)(bd.make_grid(grids[0]), bd.Grid(1, 0, 7, 1, 1, 0, 0, 0))
    assert ro(g=bad) == I and ro(b=0, g=None) == OK

    F = C.c_void_p(0x1000)
    fs = off(16, 3, 50)
    def front(hidden=F, dt=1, b=2, o=off(0, 288, 378), dim=64, pos=F, g=gs, f=fs, aq=F, sc=F, kept=F, hc=F, pc=F, si=F):
        return L.civic_compact_prefill_ragged(hidden, dt, b, P(o), dim, pos, g, P(f), aq, C.c_float(1.0), sc, kept, hc, pc, si, None)
    assert front(dt=7) == I and front(dim=0) == I and front(o=None) == I and front(o=off(0, 100, 378)) == I and front(g=None) == I
    assert front(f=None) == I and front(hidden=None) == I and front(aq=None) == I and front(sc=None) == I and front(kept=None) == I
    assert front(hc=None) == I and front(pc=None) == I and front(si=None) == I and front(pos=None) == I
    assert front(f=off(16, 3, 30)) == I                              # second sample: overlapping frames (3 + 35 > 30)
    assert front(f=off(40, 3, 50)) == I                              # first sample: the frame runs past its rows
    assert front(dim=60) == I                                        # rows that are not whole 16-byte pieces
    assert front(b=0, o=off(0), g=None, f=None, hidden=None) == OK

    st = (C.c_int64 * 3)(0, 512, 128)
    def attn(q=F, k=F, o=F, b=2, ro_=off(0, 5, 12), hq=4, hkv=2, d=128, qs=st, ks=st, causal=1, kc=None, vc=None, smax=0, pos0=0, dt=1):
        return L.civic_prefill_attn_ragged(q, k, k, o, dt, b, P(ro_), hq, hkv, d, qs, ks, st, causal, C.c_float(0.0), kc, vc, smax, pos0, None)
    assert attn(ro_=None) == I and attn(ro_=off(1, 5, 12)) == I and attn(ro_=off(0, 5, 5)) == I and attn(q=None) == I and attn(k=None) == I
    assert attn(o=None) == I and attn(hq=3) == I and attn(d=60) == I and attn(qs=None) == I and attn(dt=5) == I and attn(b=-1) == I
    assert attn(kc=F) == I and attn(vc=F) == I                        # one cache without the other
    assert attn(kc=F, vc=F, smax=6) == I                              # the longest sample (7 rows) does not fit
    assert attn(kc=F, vc=F, smax=16, pos0=10) == I and attn(kc=F, vc=F, smax=16, pos0=-1) == I
    assert attn(b=0, ro_=None) == OK and attn(d=512, qs=(C.c_int64 * 3)(0, 2048, 512), ks=(C.c_int64 * 3)(0, 1024, 512)) == bd.ERR_UNSUPPORTED
    assert bd.lib.civic_last_hip_error() == 0


def test_ragged_decode_argument_errors(bd):
    L, F = bd.lib, C.c_void_p(0x1000)
    I, OK = bd.ERR_INVALID_ARG, bd.CIVIC_OK
    ctx = lambda *v: np.asarray(v, dtype=np.int32)
    P = lambda a: C.c_void_p(a.ctypes.data) if a is not None else None
    def dec(q=F, kc=F, vc=F, o=F, dt=1, b=3, n=ctx(5, 938, 17), hq=32, hkv=8, d=128, smax=1000, scale=0.0, ws=F, wsb=1 << 30):
        return L.civic_decode_attn_ragged(q, kc, vc, o, dt, b, P(n), hq, hkv, d, smax, C.c_float(scale), ws, wsb, None)
    assert dec(n=None) == I and dec(n=ctx(5, 0, 17)) == I and dec(n=ctx(5, 1001, 17)) == I and dec(n=ctx(-1, 2, 3)) == I
    assert dec(q=None) == I and dec(kc=None) == I and dec(vc=None) == I and dec(o=None) == I and dec(dt=4) == I and dec(b=-1) == I
    assert dec(hq=30) == I and dec(d=60) == I and dec(scale=-1.0) == I and dec(q=C.c_void_p(0x1004)) == I
    assert dec(d=1024) == bd.ERR_UNSUPPORTED and dec(b=0, n=None, q=None) == OK
    need = L.civic_decode_attn_ragged_workspace_bytes(1, 3, P(ctx(5, 938, 17)), 32, 8, 128)
    assert need == L.civic_decode_attn_workspace_bytes(1, 3, 32, 8, 128, 938) > 0      # laid out for the longest context
    assert dec(ws=None, wsb=0) == bd.ERR_WORKSPACE and dec(wsb=need - 1) == bd.ERR_WORKSPACE
    assert L.civic_decode_attn_ragged_workspace_bytes(1, 3, P(ctx(5, 0, 17)), 32, 8, 128) == 0
    assert bd.lib.civic_last_hip_error() == 0


def test_header_is_plain_c(tmp_path):
    """include/civic.h is a C ABI: it compiles as C99 and as C++ with nothing but the standard headers."""
    import subprocess
    src = tmp_path / "use_header.c"
    src.write_text('#include "civic.h"\nint main(void) { return CIVIC_OK; }\n')
    inc = os.path.join(ROOT, "include")
    for cmd in (["gcc", "-std=c99", "-Wall", "-Wextra", "-pedantic", "-Werror"], ["g++", "-std=c++17", "-x", "c++", "-Wall", "-Wextra", "-pedantic"]):
        r = subprocess.run(cmd + ["-I", inc, "-fsyntax-only", str(src)], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr


def test_decode_workspace_holds_four_workgroups_per_unit(bd):
    """The decode workspace has room for 1024 workgroups of up to 8 query heads (4 from 3 to 7 heads per KV head) and no more,
    whichever kernel a head grouping takes: fewer calls would fit the array of civic_decode_attn_noalloc otherwise."""
    bf16 = __import__("torch").bfloat16
    for group in range(1, 34):
        block = 8 if group >= 8 else 4 if group > 2 else group
        for batch, hkv, d, n in ((1, 1, 128, 4000), (7, 4, 128, 900), (60, 16, 32, 3315), (100, 8, 128, 268), (228, 4, 128, 8460)):
            pairs = batch * hkv * -(-group // block)
            splits = -(-1024 // pairs)
            need = bd.civic_decode_attn_workspace_bytes(bf16, batch, group * hkv, hkv, d, n)
            assert need <= (4 * batch * group * hkv * (d + 2) * splits if splits > 1 else 0), (group, batch, hkv, d, n)


def test_a_single_number_is_an_array_of_one_entry(bd):
    """Frame starts of one frame and the context of one sample may come as a plain number or a 0-d array: such a call gets past
    the shape check, to the tensors (which are on the CPU here)."""
    torch = __import__("torch")
    hidden = torch.zeros((1, 20, 8), dtype=torch.bfloat16)
    q, cache = torch.zeros((1, 2, 8), dtype=torch.bfloat16), torch.zeros((1, 2, 4, 8), dtype=torch.bfloat16)
    for kind in (int, lambda v: np.array(v, dtype=np.int64), lambda v: np.array(v, dtype=np.int32), lambda v: np.array([v], dtype=np.int64)):
        with pytest.raises(ValueError, match="device tensor"):
            bd.civic_score_visual(hidden, (1, 4, 4, 2, 2, 1, 0, 5), kind(2), torch.zeros(8), 1.0)
        with pytest.raises(ValueError, match="device tensor"):
            bd.civic_decode_attn_ragged(q, cache, cache, kind(3))
    with pytest.raises(ValueError, match="one entry per frame"):
        bd.civic_score_visual(hidden, (1, 4, 4, 2, 2, 1, 0, 5), np.zeros((1, 1), dtype=np.int64), torch.zeros(8), 1.0)


def test_attention_sizes_reach_the_kernel_they_are_chosen_for(bd):
    """The GPU tests' sizes against the host's choice of a launch: workgroups of 8 wavefronts with two row tiles each (9), of 8 or 4."""
    from test_gpu_parity import TWO_ROW_TILES
    for b, s, hq, hkv, d in TWO_ROW_TILES:
        assert bd.lib.civic_attn_workgroup(b, s, s, hq, hkv, d, 1) == 9, (b, s, hq, hkv, d)
    tiles = [(-(-s // (256 // hpb)), s % (256 // hpb) == 0, hpb, d) for b, s, hq, hkv, d in TWO_ROW_TILES
             for hpb in [4 if hq // hkv % 4 == 0 else 2 if hq // hkv % 2 == 0 else 1]]
    assert {(n % 2, full) for n, full, _, _ in tiles} == {(0, True), (0, False), (1, True), (1, False)}
    assert {hpb for _, _, hpb, _ in tiles} == {1, 2, 4} and {d for *_, d in tiles} == {72, 96, 128}
    from test_gpu_kernel_edges import EIGHT_AND_FOUR, FOUR_AND_FOUR

    def wavefronts(batch, case):
        _, s, hq, hkv, d, causal, _ = case
        return bd.lib.civic_attn_workgroup(batch, s, s, hq, hkv, d, int(causal))
    assert [wavefronts(c[0], c) for c in EIGHT_AND_FOUR] == [9] * 4 + [8] * 7 and [wavefronts(1, c) for c in EIGHT_AND_FOUR] == [4] * 11
    assert {wavefronts(b, c) for c in FOUR_AND_FOUR for b in (1, c[0])} == {4}


def test_attention_launch_of_narrow_causal_heads_is_not_modelled(bd):
    """Causal heads of up to 64 channels take workgroups of 4 wavefronts whatever the size: a new prompt length costs no model of the
    launch on the host, which wider heads need (tens of microseconds, forty times as much)."""
    import time
    rng = np.random.default_rng(3)
    sizes = [(int(b), int(s)) for b, s in zip(rng.integers(1, 40, 300), rng.integers(100, 4000, 300))]

    def pass_over(d):
        t = time.perf_counter()
        got = {bd.lib.civic_attn_workgroup(b, s, s, 32, 8, d, 1) for b, s in sizes}
        return time.perf_counter() - t, got
    narrow, wide = min(pass_over(64) for _ in range(3)), min(pass_over(128) for _ in range(3))
    assert narrow[1] == {4} and wide[1] == {4, 8, 9}
    assert narrow[0] < wide[0] / 4


def decode_shape(bd, dtype, batch, hq, hkv, d, ctx):
    """(wavefronts of a workgroup, query heads a pass, passes, splits, matrix cores); ctx: one length, or (lowest, highest) of samples
    that each have their own."""
    ragged = isinstance(ctx, tuple)
    n = np.linspace(ctx[0], ctx[1], batch).round().astype(np.int32) if ragged else np.array([ctx], dtype=np.int32)
    shape = (C.c_int32 * 5)()
    assert bd.lib.civic_decode_shape(bd.CIVIC_F32 if dtype == "fp32" else bd.CIVIC_BF16, batch, n.ctypes.data_as(C.c_void_p), int(ragged),
                                     hq, hkv, d, shape) == 0
    return tuple(shape)


@pytest.mark.parametrize("dtype,batch,hq,hkv,d,ctx,whole", [
    # as many pairs as units, or nearly: one wide workgroup for each
    ("bf16", 24, 32, 8, 128, 600, True), ("bf16", 32, 16, 8, 128, 2400, True), ("bf16", 24, 32, 8, 128, (1000, 1300), True),
    ("fp32", 28, 32, 8, 128, 2500, True), ("fp32", 51, 32, 4, 128, 2500, True), ("fp32", 24, 32, 8, 128, 1500, True),
    ("fp32", 28, 28, 4, 128, 2500, True), ("fp32", 14, 56, 8, 128, 2500, True), ("fp32", 24, 28, 4, 128, 800, True),
    ("fp32", 26, 28, 4, 128, (600, 900), True), ("fp32", 48, 32, 4, 64, (1600, 2000), True), ("bf16", 28, 16, 8, 128, (1000, 1300), True),
    ("fp32", 48, 32, 4, 128, (300, 600), False), ("fp32", 24, 64, 4, 128, (300, 600), False), ("fp32", 24, 32, 8, 128, (300, 600), True),
    # 192 workgroups with 4 or 8 heads a pass leave a quarter of the units idle for long
    ("fp32", 48, 32, 4, 128, 2000, False), ("bf16", 24, 32, 8, 256, 2000, False), ("fp32", 24, 32, 8, 128, 2000, False),
    ("fp32", 12, 56, 8, 128, 1500, False),
    # passes that share an XCD's L2 only where the contexts are cut
    ("fp32", 24, 28, 4, 128, 2500, False), ("fp32", 24, 28, 4, 64, 3000, False), ("fp32", 32, 28, 4, 128, 1000, False),
    ("fp32", 31, 28, 4, 128, 500, False), ("fp32", 26, 28, 4, 128, (1600, 2000), False)])
def test_decode_of_whole_contexts_in_wide_workgroups(bd, dtype, batch, hq, hkv, d, ctx, whole):
    """192 to 256 (sample, KV head, pass) workgroups: contexts whole in wide ones, but not where cut contexts were measured faster."""
    waves, _, _, splits, _ = decode_shape(bd, dtype, batch, hq, hkv, d, ctx)
    assert (waves > 4 and splits == 1) if whole else (waves == 4 and splits > 1)


def test_decode_of_different_lengths_whole_in_narrow_workgroups(bd):
    """One or two heads a pass and as many pairs as units: contexts within a few hundred rows of each other are whole, and narrow."""
    assert decode_shape(bd, "bf16", 32, 16, 8, 128, (300, 600))[::3] == (4, 1)
    assert decode_shape(bd, "fp32", 32, 16, 8, 64, (1000, 1300))[::3] == (4, 1)


@pytest.mark.parametrize("dtype,batch,hq,hkv,d,ctx,heads", [
    ("bf16", 1, 16, 8, 128, 469, True), ("bf16", 16, 16, 8, 128, 768, True), ("bf16", 8, 32, 8, 128, 512, True), ("bf16", 8, 32, 8, 128, 513, False),
    ("bf16", 8, 32, 8, 128, (500, 768), True), ("bf16", 8, 32, 8, 128, (500, 769), False), ("fp32", 8, 32, 1, 128, 384, True),
    ("fp32", 1, 32, 4, 128, 384, True), ("bf16", 1, 32, 1, 128, 512, True), ("fp32", 16, 16, 4, 128, 270, True),
    # the group's rows into several L2s, and too many of them
    ("bf16", 16, 16, 1, 128, 420, False), ("bf16", 32, 8, 1, 128, 400, False), ("bf16", 64, 4, 1, 128, 700, False), ("bf16", 9, 28, 4, 128, 600, False),
    ("fp32", 16, 16, 4, 128, 384, False), ("fp32", 64, 4, 1, 128, 270, False), ("bf16", 128, 2, 1, 128, 768, False),
    ("bf16", 16, 16, 1, 128, (100, 500), True), ("bf16", 16, 16, 1, 128, (500, 768), False), ("bf16", 8, 32, 4, 128, (500, 768), False),
    ("bf16", 4, 64, 4, 128, (500, 768), True), ("fp32", 8, 8, 1, 128, 256, True), ("fp32", 8, 8, 1, 128, 257, False)])
def test_decode_in_a_workgroup_for_each_query_head(bd, dtype, batch, hq, hkv, d, ctx, heads):
    """Short contexts of up to 256 query heads: a workgroup of 16 wavefronts for each, but not where the KV heads' rows would be
    fetched into several XCDs' L2s for more than the second launch costs, nor for long contexts that matrix cores would take."""
    waves, per_pass, passes, splits, _ = decode_shape(bd, dtype, batch, hq, hkv, d, ctx)
    assert ((waves, per_pass, passes, splits) == (16, 1, hq // hkv, 1)) == heads


def test_decode_sizes_reach_the_workgroups_they_are_chosen_for(bd):
    """The GPU tests' sizes against the host's choice: (wavefronts, query heads a pass, whether on the matrix cores), lanes to a row."""
    from test_gpu_kernel_edges import DECODE_CUTS, DECODE_WIDE

    def shapes(cases):
        got = set()
        for batch, hq, hkv, d, ctx, dtype in cases:
            n = np.array(ctx * batch if len(ctx) == 1 else ctx, dtype=np.int32)
            shape = (C.c_int32 * 5)()
            assert bd.lib.civic_decode_shape(bd.CIVIC_F32 if dtype == "fp32" else bd.CIVIC_BF16, batch, n.ctypes.data_as(C.c_void_p), 1,
                                             hq, hkv, d, shape) == 0
            lanes = 8
            while lanes * 16 < d * (4 if dtype == "fp32" else 2):
                lanes *= 2
            got.add((shape[0], shape[1], shape[4], lanes))
        return got
    wide, narrow = shapes(DECODE_WIDE), shapes(DECODE_CUTS)
    assert {s[:3] for s in wide} >= {(16, 1, 0), (16, 2, 0), (8, 4, 0), (8, 8, 0), (8, 4, 1), (4, 4, 1), (4, 8, 1), (4, 4, 0)}
    assert {s[3] for s in wide if s[0] == 16} == {8, 16, 32, 64}
    assert {s[:3] for s in narrow if s[0] == 4} >= {(4, 1, 0), (4, 2, 0), (4, 4, 0), (4, 8, 0), (4, 4, 1)}
    assert {s[3] for s in narrow if s[0] == 4 and s[2] == 0} == {8, 16, 32, 64}


@pytest.mark.parametrize("rows,keys,hq,hkv,d,shifted", [
    # the row tiles of a long item on few units: every fourth begins with the next item
    ((500, 61, 2700, 90, 1200, 333, 800, 60), 0, 16, 8, 128, 1), ((500, 61, 2700, 90, 1200, 333, 800, 60), 0, 16, 4, 128, 1),
    ((938, 117, 117, 938, 500, 300, 200, 800), 0, 32, 8, 128, 1), ((1365, 341, 85, 1024, 600, 341, 1365, 85), 256, 16, 16, 72, 1),
    # few heads and items of different length on some XCDs only
    ((294, 1197, 384, 157), 0, 16, 4, 72, 1), ((1732, 1357, 1609, 173), 0, 16, 16, 128, 1),
    ((1242, 274, 1044, 337, 202, 822, 1295, 133, 502, 536, 180, 271, 147, 174, 199, 507, 584, 173, 103, 243, 628, 165, 233, 173), 0, 12, 3, 128, 1),
    # the plain order has them on units of their own
    ((2000, 500, 200), 0, 16, 4, 128, 0), ((2000, 500, 200), 0, 36, 6, 64, 0), ((938, 117, 300, 650, 1500), 0, 28, 4, 64, 0),
    ((179, 51, 660, 97, 693, 1420), 512, 16, 16, 64, 0), ((937, 177, 198, 221, 192, 489, 202), 0, 8, 8, 128, 0),
    ((73, 28, 632, 75, 41, 141, 1103, 748), 256, 12, 12, 64, 0), ((1600, 1500, 1400, 1550), 512, 12, 12, 64, 0), ((400,) * 9, 0, 16, 8, 64, 0)])
def test_ragged_attention_shifts_items_where_that_spreads_the_load(bd, rows, keys, hq, hkv, d, shifted):
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    assert bd.lib.civic_attn_item_shift(len(rows), off.ctypes.data_as(C.c_void_p), keys, hq, hkv, d, int(keys == 0)) == shifted


def test_ragged_attention_sizes_reach_either_order_of_items(bd):
    from test_gpu_kernel_edges import ITEM_ORDER
    for rows, keys, hq, hkv, d, causal, shifted in ITEM_ORDER:
        off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
        got = bd.lib.civic_attn_item_shift(len(rows), off.ctypes.data_as(C.c_void_p), keys, hq, hkv, d, int(causal))
        assert got == int(shifted), (rows, keys, hq, hkv, d, got)


def test_token_weights_stay_out_of_launches_with_little_lds(bd):
    """Token weights under the second product need the LDS of its four-stage ring: from 512 output tiles on it has two, and they are a
    launch of their own, whatever else would speak for them; likewise more anchors than have a place for their factors."""
    from test_gpu_kernel_edges import TOKEN_WEIGHTS
    each = C.c_int32()
    for batch, tokens, anchors, dim, chunks in TOKEN_WEIGHTS:
        groups = bd.lib.civic_aggregate_sum_groups(batch, tokens, anchors, dim, C.byref(each))
        assert each.value == chunks and groups == -(-(-(-tokens // 64)) // chunks) * batch
    for batch in range(1, 600):
        for anchors, dim in ((100, 128), (1365, 1152), (129, 768)):
            groups = bd.lib.civic_aggregate_sum_groups(batch, 4096, anchors, dim, None)
            assert groups == 0 or batch * -(-anchors // 128) * (dim // 128) < 512
    assert bd.lib.civic_aggregate_sum_groups(1, 60000, 24 * 1024 + 1, 128, None) == 0


@pytest.mark.parametrize("batch,tokens,anchors,dim,inside", [
    (2, 4096, 1365, 1152, True), (2, 2048, 1365, 1152, True), (1, 8192, 2730, 768, True), (3, 12000, 1333, 1280, True), (4, 12000, 1333, 1152, True),
    (1, 4096, 2730, 1152, False), (1, 8192, 2730, 1152, False), (1, 8086, 2695, 1280, False), (2, 6144, 3072, 1152, False),
    (2, 6144, 4096, 768, False), (3, 8192, 4096, 128, False), (3, 12000, 1333, 768, False)])
def test_token_weights_under_the_second_product_where_that_is_faster(bd, batch, tokens, anchors, dim, inside):
    assert (bd.lib.civic_aggregate_sum_groups(batch, tokens, anchors, dim, None) > 0) == inside

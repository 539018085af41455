"""Sizes at which a kernel's tiling or a rule of its dispatch can go wrong (edges of tiles, remainders, the smallest and the
largest of a range), against the CPU oracle.  Every tolerance is derived beside its test."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from paper_2605_28115_amd import workloads as wl
from test_gpu_parity import log, to_dev, to_host, widen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bd():
    from paper_2605_28115_amd import binding
    assert torch.cuda.is_available(), "these tests need the MI355X"
    return binding


@pytest.mark.parametrize("tokens", [1, 63, 64, 65, 200])
@pytest.mark.parametrize("anchors", [1, 127, 129, 511, 513, 700])
def test_token_weight_columns_and_row_slots(bd, tokens, anchors):
    """Token weights over column groups of 64 and row slots of 128 x 4.  A weight is exp(logit) over its row's sum, logits
    are at most 1 (inv_tau = 1): operands rounded to bf16 move one by at most 2 * 2^-9, so a weight and its row's sum by
    2^-8 each, the weight's own rounding by 2^-9: 2^-6 relative covers them, and the fp32 sums' 2^-20."""
    log("token weights", tokens, anchors)
    rng = np.random.default_rng(1000 * tokens + anchors)
    x, x32 = wl.quantize(rng.standard_normal((2, tokens, 64)).astype(np.float32), "bf16")
    a, a32 = wl.quantize(rng.standard_normal((anchors, 64)).astype(np.float32), "bf16")
    _, tw = bd.civic_anchor_aggregate(to_dev(x), to_dev(a), 1.0, want_token_weight=True)
    _, ref = oracle.anchor_aggregate(x32, a32, 1.0, want_col_sum=True)
    got = to_host(tw).astype(np.float64)
    assert (np.abs(got - ref) <= 2.0 ** -6 * ref).all(), float((np.abs(got - ref) / ref).max())


def _aggregate_bar(x, anchors, inv_tau, z):
    """What bf16 leaves of Z_0's error, element by element (see test_anchor_softmax_routes)."""
    def norm(t):
        c = t.astype(np.float64) - t.mean(-1, keepdims=True, dtype=np.float64)
        n = np.sqrt((c * c).sum(-1, keepdims=True))
        return np.where(n > 0, c / np.where(n > 0, n, 1.0), 0.0)

    logit, rounding = inv_tau * 2.0 ** -9 / np.sqrt(x.shape[-1]), 2.0 ** -9 / np.sqrt(3.0)
    out = []
    for xb, zb in zip(x, z.astype(np.float64)):
        rows, which = np.unique(xb, axis=0, return_inverse=True)
        logits = inv_tau * (norm(anchors) @ norm(xb).T)
        w = np.exp(logits - logits.max(-1, keepdims=True))
        w /= w.sum(-1, keepdims=True)
        group = np.zeros((len(anchors), len(rows)))
        np.add.at(group.T, which.reshape(-1), w.T)
        rows = rows.astype(np.float64)
        g2 = group ** 2
        about_zero = g2 @ rows ** 2
        about_z = np.maximum(about_zero - 2 * zb * (g2 @ rows) + zb ** 2 * g2.sum(-1, keepdims=True), 0.0)
        out.append(8 * np.sqrt(logit ** 2 * about_z + rounding ** 2 * about_zero) + 2.0 ** -8 * np.abs(zb) + 1e-6 * np.abs(xb).max())
    return np.stack(out)


@pytest.mark.parametrize("inv_tau", [0.0, 5.0, 60.0, 60.5])
@pytest.mark.parametrize("tokens,anchors,dim", [(1, 1, 64), (63, 127, 64), (64, 128, 128), (65, 129, 64), (129, 130, 192), (700, 260, 128)])
def test_anchor_softmax_routes(bd, inv_tau, tokens, anchors, dim):
    """Both routes of the softmax (exponentials straight out of the first product up to inv_tau = 60, logits and a row pass
    above), with logits over the whole range [-inv_tau, inv_tau]: tokens that are an anchor or its negative, and tokens with a
    mean ten times their spread.  An element of Z_0 is sum w x; the weight of a token is off by its logit's error (rounding Q_A to
    bf16, 2^-9 inv_tau / sqrt(dim) at most on average, for a token that is the anchor) and by its own rounding (2^-9 / sqrt 3),
    independently of other tokens but not of equal or opposite ones: eight times the root of the squares over the distinct
    tokens, and the rounding of the result.  A logit's error leaves the sum of the weights 1 and counts by x - Z_0; a weight's own
    rounding counts by x, since above 60 the weights are rounded after the division.  (One token of 700 left out shows.)"""
    log("softmax routes", inv_tau, tokens, anchors, dim)
    rng = np.random.default_rng(int(inv_tau) + tokens + anchors)
    a = rng.standard_normal((anchors, dim)).astype(np.float32)
    x = rng.standard_normal((2, tokens, dim)).astype(np.float32)
    x[0, ::3] = a[np.arange(0, tokens, 3) % anchors]
    x[0, 1::3] = -a[np.arange(1, tokens, 3) % anchors]
    x[1, ::2] += 10.0
    x[1, -1] = 0.5                                               # no variance: logit zero
    x, x32 = wl.quantize(x, "bf16")
    a, a32 = wl.quantize(a, "bf16")
    z, tw = bd.civic_anchor_aggregate(to_dev(x), to_dev(a), inv_tau, want_token_weight=True)
    ref, ref_tw = oracle.anchor_aggregate(x32, a32, inv_tau, want_col_sum=True)
    got = widen(to_host(z)).astype(np.float64)
    bar = _aggregate_bar(x32, a32, inv_tau, ref)
    assert np.isfinite(got).all() and (np.abs(got - ref) <= bar).all(), float((np.abs(got - ref) / bar).max())
    rel = 2.0 ** -8 + 4 * inv_tau * 2.0 ** -9 / np.sqrt(3 * dim)
    # a token's weight is a sum over the anchors of weights that are off by `rel` of themselves, plus their rows' share
    got_tw = to_host(tw).astype(np.float64)
    assert (np.abs(got_tw - ref_tw) <= 2 * rel * np.maximum(ref_tw, 1.0)).all(), float(np.abs(got_tw - ref_tw).max())


@pytest.mark.parametrize("inv_tau", [4.0, 5.0, 7.0])
@pytest.mark.parametrize("tokens,anchors,dim", [(256, 128, 1280), (300, 100, 1152), (300, 150, 1280), (700, 233, 1152)])
def test_warm_softmax_weights_are_rounded_no_worse_than_normalised_ones(bd, inv_tau, tokens, anchors, dim):
    """Weights without their row's factor, rounded to bf16, cost no more precision than normalised ones: the error of Z_0
    against 64 bits is at most that of softmax weights rounded after the division, on tokens and anchors normalised and rounded
    to bf16.  Warm softmaxes put all weights near one another, so it matters where in a binade that is: 300 tokens are the
    best place for normalised weights (1 / 300 = 2^0.77 / 512), 256 the worst.  Both errors are norms over at least 25600
    rounded weights, which scatter by 1 / sqrt(2 * 25600) = 0.45 % each: 1 % covers the difference."""
    log("warm softmax", inv_tau, tokens, anchors, dim)
    g = torch.Generator().manual_seed(tokens + dim)
    x = torch.randn((1, tokens, dim), generator=g).bfloat16().cuda()
    a = torch.randn((anchors, dim), generator=g).bfloat16().cuda()

    def norm(t):
        c = t.double() - t.double().mean(-1, keepdim=True)
        return c / c.norm(dim=-1, keepdim=True)

    def rounded(t):
        return t.float().bfloat16().double()

    qa, k0, x64 = norm(a), norm(x[0]), x[0].double()
    ref = torch.softmax(inv_tau * (qa @ k0.t().contiguous()), -1) @ x64
    normalised = rounded(rounded(torch.softmax(inv_tau * (rounded(qa) @ rounded(k0).t().contiguous()), -1)) @ x64)
    z = bd.civic_anchor_aggregate(x, a, inv_tau, want_token_weight=True)[0][0].double()
    err, bar = float((z - ref).norm() / ref.norm()), float((normalised - ref).norm() / ref.norm())
    assert err <= 1.01 * bar, (err, bar)


@pytest.mark.parametrize("inv_tau", [4.0, 30.0, 60.0, 61.0])
@pytest.mark.parametrize("binades", [-55, 0, 40, 58])
@pytest.mark.parametrize("tokens,anchors,dim", [(70, 3, 64), (200, 130, 192)])
def test_anchor_aggregate_over_the_range_of_the_tokens(bd, tokens, anchors, dim, binades, inv_tau):
    """Z_0 is as good for tokens of any size whose squares fp32 holds: tokens times 2^binades give the result times 2^binades, for
    rows whose softmax is warm, for anchors that are a token (the largest weights) and for anchors that every token points away
    from (logits of -inv_tau throughout: the smallest).  Bound of the routes' test: the logits' errors from rounding Q_A, weights
    and results rounded to bf16, per anchor against the largest token; once more 2^-8 between two such results."""
    log("token range", tokens, anchors, dim, binades, inv_tau)
    rng = np.random.default_rng(tokens + dim)
    a = rng.standard_normal((anchors, dim)).astype(np.float32)
    x = rng.standard_normal((2, tokens, dim)).astype(np.float32)
    x[0, ::7] = a[np.arange(0, tokens, 7) % anchors]
    x[1] = -a[0] + 0.01 * x[1]
    x, x32 = wl.quantize(x, "bf16")
    a, a32 = wl.quantize(a, "bf16")
    scaled = torch.from_numpy(x32 * np.float32(2.0) ** binades).bfloat16().cuda()
    z, tw = bd.civic_anchor_aggregate(scaled, to_dev(a), inv_tau, want_token_weight=True)
    ref, ref_tw = oracle.anchor_aggregate(x32, a32, inv_tau, want_col_sum=True)
    rel = 2.0 ** -8 + 4 * inv_tau * 2.0 ** -9 / np.sqrt(3 * dim)
    got = z.float().cpu().numpy().astype(np.float64) * 2.0 ** -binades
    assert np.isfinite(got).all() and np.abs(got - ref).max() <= rel * np.abs(x32).max(), float(np.abs(got - ref).max())
    assert (np.abs(to_host(tw).astype(np.float64) - ref_tw) <= 2 * rel * np.maximum(ref_tw, 1.0)).all()


# batch, tokens, anchors, dim, times 64 columns of a workgroup (0: a launch of their own)
TOKEN_WEIGHTS = [(1, 1, 1, 128, 1), (1, 64, 5, 128, 1), (1, 65, 127, 128, 1), (1, 700, 129, 128, 1), (1, 193, 767, 128, 1), (1, 300, 768, 128, 1),
                 (1, 129, 769, 128, 1), (1, 2500, 100, 128, 1), (1, 130, 1665, 128, 1), (1, 4100, 40, 128, 1), (2, 4096, 1365, 1152, 3),
                 (4, 4100, 1000, 768, 5), (1, 20000, 700, 1152, 2)]


@pytest.mark.parametrize("batch,tokens,anchors,dim,chunks", TOKEN_WEIGHTS)
def test_token_weights_under_the_second_product(bd, batch, tokens, anchors, dim, chunks):
    """Token weights made by workgroups of the second product's launch (a few items) and by a launch of their own (so many items that the
    product fills the chip twice): the same bits, and the sums of the weights of a 64-bit softmax.  Weights are rounded to bf16 (2^-9
    each, sums of them as rounded) and logits carry the rounding of the normalised anchors, 2^-9 of at most 14: 2^-5 covers them."""
    log("token weights", batch, tokens, anchors, dim)
    items = 512 // (-(-anchors // 128) * (dim // 128)) // batch * batch + batch
    each = C.c_int32()
    assert bd.lib.civic_aggregate_sum_groups(batch, tokens, anchors, dim, C.byref(each)) > 0 and each.value == chunks
    assert bd.lib.civic_aggregate_sum_groups(items, tokens, anchors, dim, None) == 0
    g = torch.Generator(device="cuda").manual_seed(tokens + anchors)
    x0 = torch.randn((batch, tokens, dim), generator=g, device="cuda").bfloat16()
    a = torch.randn((anchors, dim), generator=g, device="cuda").bfloat16()
    z1, w1 = bd.civic_anchor_aggregate(x0, a, 14.0, True)
    zn, wn = bd.civic_anchor_aggregate(x0.repeat(items // batch, 1, 1), a, 14.0, True)
    assert torch.equal(zn[-batch:], z1) and torch.equal(wn[-batch:], w1) and torch.equal(wn[:batch], w1)

    def norm(x):
        x = x.double() - x.double().mean(-1, keepdim=True)
        return x / x.norm(dim=-1, keepdim=True)

    for x, w in zip(x0, w1):
        ref = torch.softmax(14.0 * norm(a) @ norm(x).T.contiguous(), -1).sum(0)
        assert (w.double() - ref).abs().max().item() <= 2.0 ** -5 * ref.max().item()


@pytest.mark.parametrize("seq", [1, 15, 16, 17, 31, 32, 33, 127, 128, 129, 161])
@pytest.mark.parametrize("dtype,head_dim", [("fp32", 8), ("fp32", 64), ("fp32", 72), ("fp32", 128), ("fp32", 136), ("fp32", 192),
                                            ("fp32", 256), ("bf16", 136), ("bf16", 192), ("bf16", 256)])
def test_fp32_attention_tiles(bd, seq, dtype, head_dim):
    """The fp32 matrix-core kernel around its 16 rows, 32 keys and four key streams, over its four head sizes and their
    remainders, with the cache write, masked and unmasked.  fp32 bar of the parity tests (products over 256 channels and sums
    over a few hundred keys stay at 1e-6); bf16: the output's rounding."""
    log("fp32 attention", seq, dtype, head_dim)
    rng = np.random.default_rng(seq * 1000 + head_dim)
    q, q32 = wl.quantize(rng.standard_normal((2, seq, 4, head_dim)).astype(np.float32), dtype)
    k, k32 = wl.quantize(rng.standard_normal((2, seq, 2, head_dim)).astype(np.float32), dtype)
    v, v32 = wl.quantize(rng.standard_normal((2, seq, 2, head_dim)).astype(np.float32), dtype)
    for causal in (True, False):
        kc = torch.full((2, 2, seq + 3, head_dim), 7.0, dtype=torch.float32 if dtype == "fp32" else torch.bfloat16, device="cuda")
        vc = kc.clone()
        out = bd.civic_prefill_attn_kv(to_dev(q), to_dev(k), to_dev(v), kc, vc, 2, causal)
        ref = oracle.attention(q32, k32, v32, causal)
        err = float(np.abs(widen(to_host(out)).astype(np.float64) - ref).max())
        assert err <= (1e-5 if dtype == "fp32" else 2.0 ** -8) * max(1.0, float(np.abs(ref).max())), err
        for cache, x in ((kc, k), (vc, v)):
            c = to_host(cache)
            assert (c[:, :, 2:2 + seq] == x.transpose(0, 2, 1, 3)).all()
            assert (widen(c[:, :, :2]) == 7.0).all() and (widen(c[:, :, 2 + seq:]) == 7.0).all()


@pytest.mark.parametrize("n_kv", [1, 16, 48, 63, 64, 65, 80, 128, 193])
@pytest.mark.parametrize("dtype,head_dim", [("fp32", 64), ("fp32", 128), ("fp32", 192), ("fp32", 256), ("bf16", 192), ("bf16", 256)])
def test_fp32_attention_tile_lengths(bd, n_kv, dtype, head_dim):
    """Tiles of 16 and of 32 keys on both sides of the rule between them (64 keys, 128 channels), over key counts that end on a
    tile and beside one, with another number of queries.  Bars of test_fp32_attention_tiles."""
    log("fp32 attention tiles", n_kv, dtype, head_dim)
    rng = np.random.default_rng(n_kv + head_dim)
    q, q32 = wl.quantize(rng.standard_normal((2, 19, 4, head_dim)).astype(np.float32), dtype)
    k, k32 = wl.quantize(rng.standard_normal((2, n_kv, 2, head_dim)).astype(np.float32), dtype)
    v, v32 = wl.quantize(rng.standard_normal((2, n_kv, 2, head_dim)).astype(np.float32), dtype)
    out = widen(to_host(bd.civic_cross_attn(to_dev(q), to_dev(k), to_dev(v)))).astype(np.float64)
    qq, kk, vv = (torch.from_numpy(x).double().transpose(1, 2) for x in (q32, k32, v32))
    kk, vv = kk.repeat_interleave(2, 1), vv.repeat_interleave(2, 1)
    ref = (torch.softmax((qq[:, :, :, None] * kk[:, :, None]).sum(-1) / head_dim ** 0.5, -1)[..., None] * vv[:, :, None]).sum(-2).transpose(1, 2).numpy()
    assert np.abs(out - ref).max() <= (1e-5 if dtype == "fp32" else 2.0 ** -8) * max(1.0, float(np.abs(ref).max()))


@pytest.mark.parametrize("batch,seq,q_heads,kv_heads", [
    (1, 513, 16, 8), (1, 130, 28, 4), (3, 97, 7, 7), (2, 255, 9, 1), (1, 1000, 8, 8), (1, 17, 200, 4), (1, 2000, 5, 1),
    (4, 257, 16, 8), (1, 40, 300, 3)])
def test_fp32_attention_order_of_row_tiles(bd, batch, seq, q_heads, kv_heads):
    """Every row tile of every head and sample is computed once, whatever the passes over the units: one and several of them, whole
    and not, units that do not divide by the heads, and launches that take none.  fp32 bar of the parity tests."""
    log("fp32 attention, order", batch, seq, q_heads, kv_heads)
    g = torch.Generator().manual_seed(seq + q_heads)
    q, k, v = (torch.randn((batch, seq, n, 64), generator=g) for n in (q_heads, kv_heads, kv_heads))
    out = torch.full(q.shape, float("nan"), device="cuda")
    bd.civic_prefill_attn(q.cuda(), k.cuda(), v.cuda(), True, out=out)
    qq, kk, vv = (x.double().transpose(1, 2) for x in (q, k, v))
    kk, vv = (x.repeat_interleave(q_heads // kv_heads, 1) for x in (kk, vv))
    z = torch.matmul(qq, kk.transpose(2, 3)) / 8.0
    z.masked_fill_(torch.ones(seq, seq, dtype=torch.bool).triu(1), float("-inf"))
    ref = torch.matmul(torch.softmax(z, -1), vv).transpose(1, 2)
    assert (out.cpu().double() - ref).abs().max().item() <= 1e-5 * max(1.0, ref.abs().max().item())


def test_fp32_attention_more_row_tiles_than_a_grid_has(bd):
    """65535 row tiles of 16 rows and some more, two samples: weights over three keys, fp32 bar of the parity tests."""
    n = 65535 * 16 + 21
    log("fp32 attention, rows", n)
    g = torch.Generator(device="cuda").manual_seed(5)
    q = torch.randn((2, n, 2, 8), generator=g, device="cuda")
    k, v = (torch.randn((2, 3, 1, 8), generator=g, device="cuda") for _ in range(2))
    out = torch.full(q.shape, float("nan"), device="cuda")
    bd.civic_cross_attn(q, k, v, out=out)
    z = (q[:, :, :, None] * k[:, None, None, :, 0]).sum(-1) / 8 ** 0.5
    ref = (torch.softmax(z, -1)[..., None] * v[:, None, None, :, 0]).sum(-2)
    assert (out - ref).abs().max().item() <= 1e-5 * max(1.0, ref.abs().max().item())


@pytest.mark.parametrize("seq,at", [(17, 16), (40, 33), (64, 50), (150, 149)])
@pytest.mark.parametrize("head_dim", [64, 72, 256])
def test_fp32_attention_hidden_rows_hold_anything(bd, seq, at, head_dim):
    """Under the causal mask a row's result does not depend on later rows of V, whatever they hold: the rows before `at` are
    bit for bit what finite rows give, and the rows that see an infinity or NaN in a channel return it there."""
    log("fp32 attention, odd values", seq, at, head_dim)
    g = torch.Generator().manual_seed(seq + head_dim)
    q, k, v = (torch.randn((1, seq, n, head_dim), generator=g).cuda() for n in (4, 2, 2))
    clean = bd.civic_prefill_attn(q, k, v, True)
    v[:, at, :, 3], v[:, at, :, 6], v[:, at, :, head_dim - 1] = float("nan"), float("inf"), float("-inf")
    got = bd.civic_prefill_attn(q, k, v, True)
    assert torch.equal(got[:, :at], clean[:, :at])
    seen = got[:, at]
    assert torch.isnan(seen[..., 3]).all() and (seen[..., 6] == float("inf")).all() and (seen[..., head_dim - 1] == float("-inf")).all()
    keep = [c for c in range(head_dim) if c not in (3, 6, head_dim - 1)]
    assert torch.equal(got[..., keep], clean[..., keep])


@pytest.mark.parametrize("seq", [1, 16, 45])
@pytest.mark.parametrize("dtype,head_dim", [(torch.float32, 8), (torch.float32, 24), (torch.float32, 72), (torch.float32, 136),
                                            (torch.float32, 256), (torch.bfloat16, 8), (torch.bfloat16, 136)])
def test_fp32_attention_reads_its_own_rows_only(bd, dtype, head_dim, seq):
    """The fp32 matrix-core kernel where a row is shorter than, or ends inside, the 16 channels of a matrix step: Q, K, V and
    the output are parts of larger tensors whose other elements (the channels after a row, which are the next head's or the next
    key's front in a dense tensor, and whatever follows the last row) are NaN, so a read past a row that reaches a product, and a
    write past one, shows.  bf16 at 8 channels comes here with rotary positions (the bf16 kernel has no such head).  The result
    is bit for bit that of dense tensors."""
    log("fp32 attention, own rows", dtype, head_dim, seq)
    g = torch.Generator().manual_seed(seq + head_dim)
    q, k, v = (torch.randn((1, seq, n, head_dim), generator=g).cuda().to(dtype) for n in (4, 2, 2))
    angle = torch.rand((1, seq, head_dim // 2), generator=g)
    cs = torch.stack([torch.cos(angle), torch.sin(angle)], -1).cuda().contiguous()

    def inside(t):
        wide = torch.full((1, seq + 1, t.shape[2] + 1, head_dim + 8), float("nan"), dtype=dtype, device="cuda")
        part = wide[:, :seq, :t.shape[2], :head_dim]
        part.copy_(t)
        return wide, part

    def run(q, k, v, causal, out):
        if dtype == torch.bfloat16 and head_dim == 8:
            return bd.civic_prefill_attn_rope(q, k, v, cs, causal, out=out)
        return bd.civic_prefill_attn(q, k, v, causal, out=out)

    for causal in (True, False):
        dense = run(q, k, v, causal, torch.empty_like(q))
        wide, out = inside(q)
        got = run(inside(q)[1], inside(k)[1], inside(v)[1], causal, out)
        assert torch.isfinite(dense).all() and torch.equal(got, dense)
        out.fill_(float("nan"))
        assert torch.isnan(wide).all()
    # a key that a row does not see changes nothing, and an infinite channel that the query weighs with zero keeps to its own key
    clean = run(q, k, v, True, torch.empty_like(q))
    k[:, seq - 1, :, :] = float("nan")
    odd = run(q, k, v, True, torch.empty_like(q))
    assert torch.equal(odd[:, :seq - 1], clean[:, :seq - 1]) and torch.isnan(odd[:, seq - 1]).all()


@pytest.mark.parametrize("seq", [17, 40, 70])
@pytest.mark.parametrize("head_dim", [8, 24, 72, 128, 136])
def test_fp32_attention_key_of_minus_infinity_weighs_nothing(bd, head_dim, seq):
    """A logit of minus infinity is a weight of zero, at every head size: a K row holds -infinity in a channel where all queries
    are positive (the first one, which steps past the end of a row used to read again).  Against the same call without that key:
    the sums over the other keys run in another order, fp32 bar of the parity tests."""
    log("fp32 attention, minus infinity", head_dim, seq)
    g = torch.Generator().manual_seed(seq * 3 + head_dim)
    q, k, v = (torch.randn((1, seq, n, head_dim), generator=g).cuda() for n in (4, 2, 2))
    q[..., 0] = q[..., 0].abs() + 0.1
    at = seq // 2
    k[:, at, :, 0] = float("-inf")
    got = bd.civic_prefill_attn(q, k, v, False)
    keep = [i for i in range(seq) if i != at]
    ref = bd.civic_cross_attn(q, k[:, keep].contiguous(), v[:, keep].contiguous())
    assert torch.isfinite(got).all() and float((got - ref).abs().max()) <= 1e-5 * max(1.0, float(ref.abs().max()))


@pytest.mark.parametrize("batch,hq,hkv,d,ctx", [
    (1, 8, 8, 128, [1]), (1, 4, 1, 128, [64]), (1, 4, 1, 128, [65]), (3, 4, 2, 128, [1, 700, 64]), (2, 8, 1, 64, [9000, 3]),
    (60, 8, 8, 64, [40 + 7 * i for i in range(60)]), (52, 8, 8, 32, [1 + 97 * i for i in range(52)]), (48, 16, 8, 128, [300] * 48),
    (260, 2, 2, 64, [1 + i % 130 for i in range(260)]),
    # the matrix-core kernel: 3 to 17 heads per KV head, channels that are not whole chunks, steps of 32 and rounds of 128
    (2, 6, 2, 40, [31, 33]), (1, 16, 1, 128, [257]), (1, 17, 1, 128, [129]), (2, 33, 1, 72, [127, 600]), (3, 12, 4, 96, [1, 128, 385]),
    (70, 18, 6, 8, [20 * i + 1 for i in range(70)]),
    # the most LDS: eight heads of 512 channels on the vector kernel, sixteen of 128 on the matrix cores
    (1, 8, 1, 512, [70]), (2, 24, 3, 256, [300, 45]), (1, 32, 2, 128, [700])])
def test_decode_cuts(bd, batch, hq, hkv, d, ctx):
    """How a decode launch is cut: one piece per sample and several, samples of one piece beside samples of many, pieces that
    end on a round and one row past it, more than one group of samples, up to 8 splits and more.  Rows past a context are NaN.
    bf16 rounds the result once (2^-9 of it; weighted means of values that are bf16 already)."""
    log("decode cuts", batch, hq, hkv, d, max(ctx))
    rng = np.random.default_rng(sum(ctx))
    q = wl.quantize(rng.standard_normal((batch, hq, d)).astype(np.float32), "bf16")[0]
    kc, vc = (wl.quantize(rng.standard_normal((batch, hkv, max(ctx) + 1, d)).astype(np.float32), "bf16")[0] for _ in range(2))
    for b, n in enumerate(ctx):
        kc[b, :, n:] = 0x7FC0
        vc[b, :, n:] = 0x7FC0
    outs = [bd.civic_decode_attn_ragged(to_dev(q), to_dev(kc), to_dev(vc), ctx)]
    if len(set(ctx)) == 1:
        outs.append(bd.civic_decode_attn(to_dev(q), to_dev(kc), to_dev(vc), ctx[0]))
    for out in outs:
        got = widen(to_host(out)).astype(np.float64)
        for b, n in enumerate(ctx):
            ref = oracle.decode_attention(widen(q[b:b + 1]), widen(kc[b:b + 1]), widen(vc[b:b + 1]), n)
            assert np.abs(got[b] - ref[0]).max() <= 2.0 ** -8 * max(1.0, float(np.abs(ref).max())), (b, n)


def _decode_reference(q, k, v, n):
    """Softmax attention of one query per head over the first n rows, in 64 bits; an infinite logit and an infinity in V are
    what the formula makes of them."""
    hq, hkv = q.shape[1], k.shape[1]
    qg, kk, vv = q.double().view(q.shape[0], hkv, hq // hkv, -1), k[:, :, :n].double(), v[:, :, :n].double()
    logits = (qg[:, :, :, None, :] * kk[:, :, None]).sum(-1) / q.shape[-1] ** 0.5
    p = torch.softmax(logits, -1)
    return (p[..., None] * vv[:, :, None]).sum(-2).view(q.shape)


DECODE_GROUPS = [(2, 1), (4, 1), (4, 2), (16, 1), (17, 1), (6, 2)]


@pytest.mark.parametrize("hq,hkv", DECODE_GROUPS)
@pytest.mark.parametrize("d,n", [(8, 40), (40, 33), (64, 200), (72, 300), (128, 64), (128, 1500)])
def test_decode_keys_of_minus_infinity_weigh_nothing(bd, hq, hkv, d, n):
    """Logits of minus infinity, with one and two heads per KV head (vector kernel) and more (matrix cores), in one piece and in
    several: a single key, the whole first 32 keys (a wavefront that has met no weight yet) and a whole piece weigh nothing, at
    head sizes that are not whole steps of 32 channels too; no key with a weight at all is 0 / 0.  bf16 rounds the result once."""
    log("decode, minus infinity", hq, hkv, d, n)
    g = torch.Generator().manual_seed(hq + 10 * d + n)
    q, k, v = (torch.randn((2, h, *s, d), generator=g).bfloat16() for h, s in ((hq, ()), (hkv, (n,)), (hkv, (n,))))
    q[..., 0] = q[..., 0].abs() + 0.25
    for hidden in ((5,), tuple(range(32)), tuple(range(n - 1)), tuple(range(n))):
        kk = k.clone()
        kk[:, :, list(hidden), 0] = float("-inf")
        got = bd.civic_decode_attn(q.cuda(), kk.cuda(), v.cuda(), n).cpu().double()
        if len(hidden) == n:
            assert torch.isnan(got).all()
            continue
        ref = _decode_reference(q, kk, v, n)
        assert torch.isfinite(got).all() and float((got - ref).abs().max()) <= 2.0 ** -8 * max(1.0, float(ref.abs().max()))


@pytest.mark.parametrize("hq,hkv", DECODE_GROUPS)
@pytest.mark.parametrize("d,n,at", [(8, 40, 39), (40, 33, 32), (64, 200, 0), (72, 300, 150), (128, 64, 63), (128, 1500, 700), (128, 1500, 1499)])
def test_decode_infinities_of_v_stay_what_they_are(bd, hq, hkv, d, n, at):
    """An infinity or NaN in a row of V is the result in its channel (every weight here is far from zero), at one and two heads
    per KV head and at more alike, in the last row too (which keys past the end read again); all other channels, and rows past
    the context, whatever they hold, change nothing.  bf16 rounds the result once."""
    log("decode, infinities of V", hq, hkv, d, n, at)
    g = torch.Generator().manual_seed(hq + 10 * d + n)
    q, k, v = (torch.randn((2, h, *s, d), generator=g).bfloat16() for h, s in ((hq, ()), (hkv, (n + 2,)), (hkv, (n + 2,))))
    k[:, :, n:], v[:, :, n:] = float("nan"), float("inf")
    v[:, :, at, 3], v[:, :, at, 6], v[:, :, at, d - 1] = float("nan"), float("inf"), float("-inf")
    ref = _decode_reference(q, k, v, n)
    outs = [bd.civic_decode_attn(q.cuda(), k.cuda(), v.cuda(), n), bd.civic_decode_attn_ragged(q.cuda(), k.cuda(), v.cuda(), [n, n])]
    for got in (o.cpu().double() for o in outs):
        assert torch.isnan(got[..., 3]).all() and (got[..., 6] == float("inf")).all() and (got[..., d - 1] == float("-inf")).all()
        keep = [c for c in range(d) if c not in (3, 6, d - 1)]
        diff = (got[..., keep] - ref[..., keep]).abs().max()
        assert float(diff) <= 2.0 ** -8 * max(1.0, float(ref[..., keep].abs().max()))


@pytest.mark.parametrize("group", [2, 4, 16])
@pytest.mark.parametrize("n", [3, 300, 2000])
def test_decode_weights_are_fp32(bd, group, n):
    """The softmax weights meet V with all bits of fp32: three rows of V cancel to about 2^-18 of themselves, so the error of the
    weights is what is left.  Against 64 bits, relative to sum p |v|: the logit's two roundings, exp2 and the factors of the merges
    (2^-23 each at logits of at most 1) and a few sums stay below 2^-20; a weight of 16 bits is off by up to 2^-18.  The output's
    rounding is 2^-9 of the small result."""
    log("decode weights", group, n)
    batch, hkv, d = 8, 4, 64
    g = torch.Generator().manual_seed(group + n)
    q = torch.zeros(batch, hkv, d)
    q[..., 0] = 1.0 + torch.rand((batch, hkv), generator=g)
    k = torch.zeros(batch, hkv, n, d)
    k[..., 0] = 4.0 * torch.rand((batch, hkv, n), generator=g)
    q, k = q.bfloat16(), k.bfloat16()
    p = torch.softmax((q[:, :, None, :1].double() * k[..., :1].double()).sum(-1) / 8.0, -1)
    at = [0, n // 2, n - 1]
    v = torch.zeros(batch, hkv, n, d, dtype=torch.float64)
    v[:, :, at[0]] = (1.0 + torch.rand((batch, hkv, d), generator=g)).bfloat16().double()
    left = p[:, :, at[0], None] * v[:, :, at[0]]
    for i in at[1:]:
        v[:, :, i] = (-left / p[:, :, i, None]).float().bfloat16().double()
        left = left + p[:, :, i, None] * v[:, :, i]
    bar = 2.0 ** -20 * (p[..., None] * v.abs()).sum(-2) + 2.0 ** -8 * left.abs()
    out = bd.civic_decode_attn(q.repeat_interleave(group, 1).cuda(), k.cuda(), v.bfloat16().cuda(), n)
    err = (out.cpu().double().view(batch, hkv, group, d) - left[:, :, None]).abs() / bar[:, :, None]
    assert float(err.max()) <= 1.0, float(err.max())


@pytest.mark.parametrize("batch,hq,hkv,d,n", [(228, 24, 4, 128, 600), (50, 112, 16, 96, 320), (100, 48, 8, 128, 268)])
def test_noalloc_takes_groups_of_five_to_seven_heads(bd, batch, hq, hkv, d, n):
    """Head groupings whose blocks of heads differ between the two decode kernels: the call without a workspace is taken where
    its array held the splits before there was a second kernel, and returns the same bits as the call with one."""
    log("noalloc", batch, hq, hkv, d, n)
    g = torch.Generator(device="cuda").manual_seed(n)
    q = torch.randn((batch, hq, d), generator=g, device="cuda").bfloat16()
    k, v = (torch.randn((batch, hkv, n, d), generator=g, device="cuda").bfloat16() for _ in range(2))
    out = torch.empty_like(q)
    bd.civic_decode_attn_noalloc(q, k, v, n, out)
    assert torch.equal(out, bd.civic_decode_attn(q, k, v, n))


DECODE_CUTS = [
    (70, 16, 4, 96, [600] * 70, "fp32"), (20, 28, 4, 64, [1100] * 20, "fp32"), (12, 14, 2, 64, [511] * 12, "fp32"),   # 4 and 8 splits, and not
    (3, 16, 2, 64, [128, 129, 300], "fp32"), (2, 8, 1, 128, [64, 65], "fp32"), (1, 9, 1, 256, [200], "fp32"),
    (33, 8, 1, 64, [128, 129, 300] * 11, "fp32"), (34, 8, 1, 128, [64, 65] * 17, "fp32"),                             # eight heads a pass
    (2, 4, 1, 32, [257, 40], "fp32"), (2, 4, 1, 36, [33, 500], "fp32"), (3, 2, 2, 64, [90, 1, 400], "bf16"),
    (66, 4, 1, 32, [257, 40] * 33, "fp32"), (66, 4, 1, 36, [33, 500] * 33, "fp32"),                                   # 8 and 4 row slots
    (3, 4, 2, 128, [90, 64, 400], "bf16"), (2, 2, 1, 512, [70, 9], "bf16"),
    (66, 4, 2, 128, [90, 64, 400] * 22, "bf16"), (130, 2, 1, 512, [70, 9] * 65, "bf16"),                              # 4 and 1
    (30, 8, 4, 128, [1 + 17 * i for i in range(30)], "fp32"), (64, 8, 4, 64, [250 + 7 * i for i in range(64)], "fp32"),  # pieces, whole
    (66, 16, 4, 72, [1100] * 66, "bf16"), (33, 32, 8, 64, [200 + i for i in range(33)], "bf16")]


@pytest.mark.parametrize("batch,hq,hkv,d,ctx,dtype", DECODE_CUTS)
def test_decode_cuts_of_either_kernel(bd, batch, hq, hkv, d, ctx, dtype):
    """The rules of the cuts that go by the kernel and its heads a pass, and both ways a workgroup's states meet.  Rows past a
    context are NaN.  fp32: bar of the parity tests; bf16 rounds the result once."""
    log("decode cuts", dtype, batch, hq, hkv, d, max(ctx))
    g = torch.Generator().manual_seed(sum(ctx))
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    q, k, v = (torch.randn((batch, h, *n, d), generator=g).to(dt) for h, n in ((hq, ()), (hkv, (max(ctx) + 1,)), (hkv, (max(ctx) + 1,))))
    ref = torch.empty((batch, hq, d), dtype=torch.float64)
    for b, n in enumerate(ctx):
        ref[b] = _decode_reference(q[b:b + 1], k[b:b + 1], v[b:b + 1], n)[0]
        k[b, :, n:], v[b, :, n:] = float("nan"), float("nan")
    outs = [bd.civic_decode_attn_ragged(q.cuda(), k.cuda(), v.cuda(), ctx)]
    if len(set(ctx)) == 1:
        outs.append(bd.civic_decode_attn(q.cuda(), k.cuda(), v.cuda(), ctx[0]))
    for out in outs:
        err = float((out.cpu().double() - ref).abs().max())
        assert err <= (1e-5 if dtype == "fp32" else 2.0 ** -8) * max(1.0, float(ref.abs().max())), err


DECODE_WIDE = [
    (1, 16, 8, 128, [257], "bf16"), (1, 16, 8, 128, [768], "bf16"), (1, 16, 8, 128, [769], "bf16"),         # three rounds of 16 wavefronts
    (8, 32, 8, 128, [300], "bf16"), (9, 32, 8, 128, [300], "bf16"), (1, 9, 1, 128, [20, ], "fp32"), (1, 9, 1, 128, [33], "fp32"),  # 256 heads
    (3, 6, 6, 72, [300, 257, 1], "bf16"), (2, 2, 1, 64, [900, 1024], "bf16"), (1, 2, 1, 256, [200], "bf16"), (2, 2, 2, 512, [100, 64], "bf16"),
    (2, 8, 4, 128, [256], "fp32"), (2, 8, 4, 128, [257, 129], "fp32"), (2, 3, 3, 32, [1000, 513], "fp32"),   # eight lanes a row
    (2, 8, 2, 64, [250, 256], "fp32"), (2, 9, 1, 64, [255], "fp32"), (1, 16, 2, 256, [63], "fp32"),
    (28, 32, 8, 64, [257], "fp32"), (25, 64, 8, 64, [129], "fp32"), (28, 28, 4, 64, [300], "fp32"),           # 8 wavefronts, 4 and 8 heads
    (28, 32, 8, 128, [170 + i for i in range(28)], "fp32"), (52, 32, 4, 128, [70 + i for i in range(52)], "fp32"),
    (32, 8, 1, 128, [400], "bf16"), (16, 16, 1, 128, [300], "bf16"), (64, 4, 1, 128, [300], "fp32"),          # rows into several L2s
    (2, 16, 1, 512, [33, 20], "bf16"), (1, 4, 1, 200, [120], "bf16"),
    (4, 28, 4, 128, [300, 320, 257, 1], "bf16"), (1, 32, 2, 128, [320], "bf16"), (1, 17, 1, 64, [257], "bf16"), (1, 32, 8, 96, [321], "bf16"),
    (96, 2, 1, 64, [600], "bf16"), (97, 2, 1, 64, [600], "bf16"), (24, 16, 4, 64, [300], "bf16"), (25, 16, 4, 64, [300], "bf16"),  # 96 pairs
    (24, 32, 8, 64, [600], "bf16"), (32, 16, 8, 64, [700], "bf16"), (33, 16, 8, 64, [700], "bf16"), (191, 4, 1, 64, [300], "bf16"),   # 192 to 256
    (5, 32, 8, 64, [40, 2000, 700, 1, 1024], "bf16"), (3, 40, 2, 64, [900, 1, 513], "bf16"), (4, 28, 4, 64, [1500, 800, 3, 40], "fp32"),  # cut: order
    (28, 16, 8, 64, [3072], "fp32"), (28, 16, 8, 64, [3073], "fp32"), (48, 8, 4, 64, [600 + 9 * i for i in range(48)], "bf16"),
    (48, 8, 4, 64, [60 + 25 * i for i in range(48)], "bf16"), (60, 16, 4, 128, [300], "fp32")]


@pytest.mark.parametrize("batch,hq,hkv,d,ctx,dtype", DECODE_WIDE)
def test_decode_wide_workgroups(bd, batch, hq, hkv, d, ctx, dtype):
    """Workgroups of 8 and of 16 wavefronts and the rule that takes them, on both sides of its edges, one length for all samples and one
    each.  Checks and bars of test_decode_cuts_of_either_kernel."""
    test_decode_cuts_of_either_kernel(bd, batch, hq, hkv, d, ctx * batch if len(ctx) == 1 else ctx, dtype)


@pytest.mark.parametrize("case", [
    # batch, grid (frames, height, width, cell, cell, cell floor, frame floor, budget), text before / between / behind, dim, rows
    (1, (1, 1, 1, 4, 4, 1, 0, 1), 0, 0, 0, 8, "random"),          # one token, one vector a row
    (2, (1, 32, 64, 4, 4, 1, 0, 700), 3, 0, 5, 64, "random"),     # 2048 tokens: the last size of 512 threads
    (2, (1, 3, 683, 4, 4, 1, 0, 700), 3, 0, 5, 64, "random"),     # 2049: the first of 1024, rows of keys that are not aligned
    (1, (2, 64, 32, 3, 2, 2, 5, 1300), 7, 9, 0, 128, "random"),   # 4096: mark words in lanes; text placed by the selection
    (1, (3, 35, 39, 4, 3, 20, 0, 4000), 0, 1, 2, 128, "random"),  # 4095, cells kept whole
    (1, (1, 17, 241, 8, 8, 1, 0, 1300), 2, 0, 0, 8, "random"),    # 4097: mark words through LDS
    (1, (2, 128, 128, 8, 8, 1, 7, 9000), 40, 30, 20, 8, "random"),  # 32768: no room for text workgroups on the same unit
    (1, (128, 2, 2, 2, 2, 1, 0, 200), 1, 1, 1, 16, "random"),     # as many frames as there can be
    (1, (1, 16, 16, 4, 4, 0, 0, 0), 4, 0, 3, 64, "random"),       # nothing kept: text only
    (1, (2, 8, 8, 4, 4, 0, 0, 1), 0, 6, 0, 64, "random"),         # one kept token among text
    (128, (1, 8, 8, 4, 4, 1, 0, 20), 3, 0, 2, 64, "random"),      # the last batch with text workgroups, the first without
    (129, (1, 8, 8, 4, 4, 1, 0, 20), 3, 0, 2, 64, "random"),
    (300, (1, 40, 60, 4, 4, 1, 0, 2300), 9, 0, 100, 8, "random"),  # more than 2^19 tokens in samples of more than 2048: two launches
    (128, (1, 64, 64, 4, 4, 1, 0, 1365), 9, 0, 100, 8, "random"),  # 2^19 tokens: one launch
    (256, (1, 32, 64, 4, 4, 1, 0, 1900), 9, 0, 2500, 8, "random"),  # two workgroups a sample: 2204 rows each, in two runs
    (257, (1, 8, 8, 4, 4, 1, 0, 20), 3, 0, 2, 64, "random"),      # more samples than units
    (130, (1, 32, 32, 4, 4, 1, 0, 341), 64, 0, 64, 512, "random"),  # three workgroups a sample by number, one for every 128 KB
    (130, (1, 32, 32, 4, 4, 1, 0, 341), 64, 0, 64, 2048, "random"),
    (1, (1, 32, 64, 4, 4, 1, 0, 700), 3, 0, 5, 64, "equal"),      # every score 0: ties by index
    (1, (1, 64, 64, 4, 4, 1, 9, 1500), 3, 0, 5, 64, "few"),       # eight distinct scores
    (1, (1, 32, 64, 4, 4, 2, 0, 700), 3, 0, 5, 64, "outlier"),    # all but two scores in one bucket
])
def test_selection_and_merge_in_one_launch(bd, case):
    """civic_compact_prefill's second launch, where every workgroup that moves rows selects for itself, against civic_select and
    civic_compact on the same scores and against the oracle's selection: whole numbers and copied rows, no tolerance."""
    batch, grid, before, between, behind, dim, rows = case
    log("selection and merge", case)
    frames, hw = grid[0], grid[1] * grid[2]
    fs = np.asarray([before + f * (hw + between) for f in range(frames)], dtype=np.int64)
    s_len = int(fs[-1]) + hw + behind
    rng = np.random.default_rng(batch + frames * hw + dim)
    hid = rng.standard_normal((batch, s_len, dim)).astype(np.float32)
    anchor = rng.standard_normal(dim).astype(np.float32) + 0.25
    if rows == "equal":
        hid[:] = 1.0
    elif rows == "few":
        hid = hid[:, rng.integers(0, 8, s_len)]
    elif rows == "outlier":
        hid = hid[:, :1] + 1e-2 * hid
        hid[:, before + 77], hid[:, before + 1000] = anchor, -anchor
    hid, _ = wl.quantize(hid, "bf16")
    d_hid = to_dev(hid)
    d_pos = torch.from_numpy(rng.integers(0, 9000, (3, batch, s_len)).astype(np.int32)).cuda()
    d_anchor = torch.from_numpy(bd.civic_anchor_normalize(anchor)).cuda()
    k = bd.civic_kept_count(grid)
    kept = torch.full((batch, k), -1, dtype=torch.int32, device="cuda")
    scores, kept, hc, pc, si = bd.civic_compact_prefill(d_hid, d_pos, grid, fs, d_anchor, 1.0, kept_idx=kept)
    kept3, _ = bd.civic_select(scores, grid)
    hc3, pc3, si3 = bd.civic_compact(d_hid, d_pos, grid, fs, kept3)
    torch.cuda.synchronize()
    assert torch.equal(kept, kept3) and torch.equal(si, si3) and torch.equal(pc, pc3)
    assert torch.equal(hc.view(torch.int16), hc3.view(torch.int16))
    some = sorted({0, batch // 2, batch - 1})
    ref, _ = oracle.select(to_host(scores)[some], grid)
    assert np.array_equal(to_host(kept)[some], ref)


@pytest.mark.parametrize("case", [
    # rows of the items, memory, width, packed, scale of R
    ([1], 1, 8, False, 1.0), ([2, 2], 3, 72, False, 1.0), ([64], 4, 128, False, 1.0), ([65, 65], 127, 136, False, 1.0),
    ([128], 128, 1152, False, 1.0), ([129], 130, 264, False, 1.0), ([256, 256, 256], 64, 120, False, 1.0), ([257], 512, 64, False, 1.0),
    ([1, 63, 64, 65, 127, 128, 129, 385], 132, 200, True, 1.0), ([5] * 70, 8, 16, True, 1.0),     # 70 items: two launches
    ([200], 132, 136, False, 1e-36), ([200], 132, 136, False, 3e35), ([300, 40], 64, 72, True, 1e-30),  # column sums at the ends of fp32
])
def test_kv_compress_tiles_and_scales(bd, case):
    """Eq. 9 over tiles of 128 x 128 in steps of 64 rows, for any scale of R.  A weight is rounded to bf16 (2^-9), their sum moves by as
    much at most, the result is rounded once more: 2^-8 of the sum of |weight x|, and 2^-8 of the result, bound the error of an element."""
    rows, mem, width, packed, scale = case
    log("kv compress", case)
    rng = np.random.default_rng(sum(rows) + mem + width)
    lead = (sum(rows),) if packed else (len(rows), rows[0])
    k, k32 = wl.quantize(rng.standard_normal(lead + (width,)).astype(np.float32), "bf16")
    v, v32 = wl.quantize(rng.standard_normal(lead + (width,)).astype(np.float32), "bf16")
    r = (rng.random((lead[0] if packed else rows[0], mem)) ** 4 * scale).astype(np.float32)
    if mem > 2 and scale == 1.0:
        r[:, 1] = 0.0                                          # a column that weighs nothing
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    dk, dv, dr = to_dev(k), to_dev(v), torch.from_numpy(r).cuda()
    kc, vc = bd.civic_kv_compress_ragged(dk, dv, dr, off) if packed else bd.civic_kv_compress(dk, dv, dr)
    torch.cuda.synchronize()
    for got, x in ((kc, k32), (vc, v32)):
        got = widen(to_host(got)).astype(np.float64)
        for i in range(len(rows)):
            xi = x[off[i]:off[i + 1]] if packed else x[i]
            ri = (r[off[i]:off[i + 1]] if packed else r).astype(np.float64)
            total = ri.sum(0)
            w = np.where(total != 0, ri / np.where(total != 0, total, 1.0), 0.0)
            ref = w.T @ xi.astype(np.float64)
            bar = 2.0 ** -8 * (w.T @ np.abs(xi.astype(np.float64))) + 2.0 ** -8 * np.abs(ref) + 1e-30
            assert (np.abs(got[i] - ref) <= bar).all(), float((np.abs(got[i] - ref) / bar).max())


@pytest.mark.parametrize("items,rows", [(1, 1025), (1, 2048), (17, 1025), (6, 897), (3, 64), (40, 64), (30, 200), (1, 200)])
def test_kv_compress_of_a_batch_is_that_of_its_items(bd, items, rows):
    """Every item's sums run over its rows in order: the same bits in a batch, alone and packed among longer ones."""
    log("kv compress batch", items, rows)
    g = torch.Generator(device="cuda").manual_seed(items + rows)
    k = torch.randn((items, rows, 264), generator=g, device="cuda").bfloat16()
    v = torch.randn((items, rows, 264), generator=g, device="cuda").bfloat16()
    r = torch.rand((rows, 132), generator=g, device="cuda") ** 4
    kc, vc = bd.civic_kv_compress(k, v, r)
    one = bd.civic_kv_compress(k[-1:].contiguous(), v[-1:].contiguous(), r)
    long = torch.randn((1500, 264), generator=g, device="cuda").bfloat16()
    packed = torch.cat([long, k[-1]])
    kp, _ = bd.civic_kv_compress_ragged(packed, packed, torch.cat([torch.rand((1500, 132), generator=g, device="cuda"), r]), [0, 1500, 1500 + rows])
    torch.cuda.synchronize()
    assert torch.equal(one[0][0], kc[-1]) and torch.equal(one[1][0], vc[-1]) and torch.equal(kp[1], kc[-1])


@pytest.mark.parametrize("rows,mem,width", [(2, 4, 8), (65, 127, 136), (200, 130, 72), (390, 132, 64), (1025, 132, 64)])
def test_kv_compress_of_signed_assignments(bd, rows, mem, width):
    """R with negative entries, some of whose column sums nearly cancel: the error stays that of weights rounded to bf16, 2^-8 of the sum
    of |weight x| and of the result, and of an fp32 sum (chains of at most 9 + 2 + 32 terms, below 2^-16 of the sum of |weight|).  A batch,
    an item of its own and an item among longer ones give the same bits."""
    log("kv compress signed", rows, mem, width)
    rng = np.random.default_rng(rows + mem + width)
    k, k32 = wl.quantize(rng.standard_normal((3, rows, width)).astype(np.float32) + 1, "bf16")
    r = rng.standard_normal((rows, mem)).astype(np.float32)
    r[:, 3] = np.abs(r[:, 3])
    r[-1, :2] = -r[:-1, :2].astype(np.float64).sum(0) + np.asarray([0.01, -0.5]) * (1 if rows > 2 else 0.1)
    dk, dr = to_dev(k), torch.from_numpy(r).cuda()
    kc, vc = bd.civic_kv_compress(dk, dk, dr)
    w = r.astype(np.float64) / r.astype(np.float64).sum(0)
    for b in range(3):
        x = k32[b].astype(np.float64)
        ref = w.T @ x
        bar = 2.0 ** -8 * (np.abs(w).T @ np.abs(x)) + (2.0 ** -8 + 2.0 ** -16 * np.abs(w).sum(0)[:, None]) * np.abs(ref) + 1e-30
        for got in (kc, vc):
            err = np.abs(widen(to_host(got[b])).astype(np.float64) - ref)
            assert (err <= bar).all(), float((err / bar).max())
    one, _ = bd.civic_kv_compress(dk[2:].contiguous(), dk[2:].contiguous(), dr)
    assert torch.equal(one[0], kc[2])
    if mem % 4 == 0:
        long = torch.ones((1500, width), device="cuda").bfloat16()
        packed = torch.cat([long, dk[2]])
        kp, _ = bd.civic_kv_compress_ragged(packed, packed, torch.cat([torch.rand((1500, mem), device="cuda"), dr]), [0, 1500, 1500 + rows])
        assert torch.equal(kp[1], kc[2])


@pytest.mark.parametrize("spread", [0, 99])
@pytest.mark.parametrize("rows,mem,width,packed", [([1], 4, 8, False), ([65], 127, 136, False), ([300, 64, 129], 64, 304, True), ([1025], 132, 1032, False), ([1088, 1088], 128, 72, False)])
def test_kv_compress_weights_are_normalised_and_then_rounded(bd, rows, mem, width, packed, spread):
    """Rbar itself, bit for bit: a column of X that is 1 in one row and 0 elsewhere brings that row's weights out, each the fp32 quotient
    rounded to bf16 once.  R holds whole numbers, of both signs in every second column, whose sums (below 2^24) are exact in any order,
    times a power of two per column: sums from 2^-99 to 2^109 and entries far from their sum cost no bit."""
    log("kv compress weights", rows, mem, width, packed, spread)
    rng = np.random.default_rng(sum(rows) + mem)
    total = sum(rows) if packed else rows[0]
    whole = rng.integers(1, 1 << 12, (total, mem))
    whole[:, 1::2] -= 2000
    whole[:, 2] = 0
    r = (whole * 2.0 ** rng.integers(-spread, spread - 11 if spread else 1, mem)).astype(np.float32)
    lead = (total,) if packed else (len(rows), total)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    x = np.zeros(lead + (width,), dtype=np.float32)
    at = [rng.integers(0, n, width) for n in rows]
    for i, rows_of in enumerate(at):
        if packed:
            x[off[i] + rows_of, np.arange(width)] = 1.0
        else:
            x[i, rows_of, np.arange(width)] = 1.0
    dx, dr = torch.from_numpy(x).cuda().bfloat16(), torch.from_numpy(r).cuda()
    kc, vc = bd.civic_kv_compress_ragged(dx, dx, dr, off) if packed else bd.civic_kv_compress(dx, dx, dr)
    for i in range(len(rows)):
        ri = r[off[i]:off[i + 1]] if packed else r
        t = ri.astype(np.float64).sum(0).astype(np.float32)
        inv = np.where(t != 0, np.float32(1) / np.where(t != 0, t, np.float32(1)), np.float32(0))
        ref = torch.from_numpy((ri * inv)[at[i]].T.copy()).bfloat16()
        for got in (kc, vc):
            assert torch.equal(got[i].cpu(), ref)


@pytest.mark.parametrize("rows,mem", [(64, 1 << 24), (1030, 1100000)])
def test_kv_compress_of_r_of_four_gigabytes(bd, rows, mem):
    """R of 4 GB and more, whose row offsets pass 32 bits of bytes within one step (2^24 columns) or over all rows: sampled columns
    against float64, with the bound of the test of tiles and scales."""
    log("kv compress, large R", rows, mem)
    width = 8
    g = torch.Generator(device="cuda").manual_seed(rows)
    x = torch.randn((1, rows, width), generator=g, device="cuda").bfloat16()
    r = torch.rand((rows, mem), generator=g, device="cuda")
    kc, _ = bd.civic_kv_compress(x, x, r)
    at = torch.cat([torch.arange(0, 130, device="cuda"), torch.arange(mem - 130, mem, device="cuda"), torch.arange(0, mem, mem // 1000, device="cuda")])
    w = r[:, at].double()
    w /= w.sum(0)
    ref = w.T @ x[0].double()
    bar = 2.0 ** -8 * (w.T @ x[0].double().abs()) + 2.0 ** -8 * ref.abs() + 1e-30
    assert ((kc[0, at].double() - ref).abs() <= bar).all()


@pytest.mark.parametrize("d", [64, 128, 192, 256, 56, 96, 120])
@pytest.mark.parametrize("seq", [15, 64, 65, 81, 130, 1023, 1025])
def test_f32_attention_whole_heads_and_tiles_of_keys(bd, d, seq):
    """fp32 attention at the tile lengths its launch chooses between (64 and 1024 keys), for heads that fill their steps of 64 channels
    and heads that do not.  Sums of up to 1025 products in another order: 1e-5, as large as the repository's fp32 tolerance."""
    log("fp32 attention tiles", d, seq)
    rng = np.random.default_rng(d + seq)
    q, k, v = (rng.standard_normal((1, seq, h, d)).astype(np.float32) for h in (4, 2, 2))
    for causal in (True, False):
        out = to_host(bd.civic_prefill_attn(to_dev(q), to_dev(k), to_dev(v), causal))
        ref = oracle.attention(q, k, v, causal)
        assert np.abs(out.astype(np.float64) - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max())


# batch, rows, query heads, KV heads, width, causal, rotary: the batch in workgroups of 8 wavefronts, with two row tiles each where marked,
# a single sample in those of 4
EIGHT_AND_FOUR = [
    (4, 938, 32, 8, 128, True, False), (4, 938, 32, 8, 128, True, True), (3, 960, 40, 10, 96, True, True), (6, 1100, 16, 8, 72, True, False),   # two
    (6, 2817, 4, 2, 128, True, False), (2, 1365, 16, 16, 72, False, False), (4, 1153, 8, 8, 128, False, False), (8, 1200, 4, 4, 64, False, False),
    (24, 1537, 4, 4, 128, False, False), (8, 1537, 8, 8, 96, False, False), (9, 767, 8, 8, 128, False, False),
]
# both in those of 4, two and more to a unit, and around the ends of their row and key tiles
FOUR_AND_FOUR = [
    (3, 1440, 16, 4, 96, True, True), (2, 1153, 8, 8, 128, False, False), (12, 1537, 4, 4, 64, False, False),
    (3, 1, 4, 2, 64, True, False), (2, 65, 4, 4, 96, True, True), (5, 129, 4, 1, 128, True, True), (2, 161, 6, 2, 80, False, False),
]


@pytest.mark.parametrize("case", EIGHT_AND_FOUR + FOUR_AND_FOUR)
def test_attention_of_a_batch_is_that_of_its_samples(bd, case):
    """Attention, with and without rotary positions and the fused cache write, of a batch and of its samples one by one and as a ragged
    batch: launches choose workgroups of 4 or 8 wavefronts by their size, and the bits are the same.  One sample against the oracle at
    the repository's tolerance for bf16."""
    batch, seq, hq, hkv, d, causal, rope = case
    log("attention by workgroup", case)
    g = torch.Generator(device="cuda").manual_seed(seq + d)
    q, k, v = (torch.randn((batch, seq, h, d), generator=g, device="cuda").bfloat16() for h in (hq, hkv, hkv))
    table = torch.rand((batch, seq, d // 2, 2), generator=g, device="cuda") if rope else None

    def attend(lo, hi):
        if rope:
            return (bd.civic_prefill_attn_rope(q[lo:hi], k[lo:hi], v[lo:hi], table[lo:hi], causal),)
        kc, vc = (torch.zeros((hi - lo, hkv, seq + 3, d), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        return bd.civic_prefill_attn_kv(q[lo:hi], k[lo:hi], v[lo:hi], kc, vc, 3, causal), kc, vc

    whole = attend(0, batch)
    for b in {0, batch - 1}:
        for x, y in zip(whole, attend(b, b + 1)):
            assert torch.equal(x[b], y[0]), b
    if not rope:
        packed = bd.civic_prefill_attn_ragged(q.flatten(0, 1), k.flatten(0, 1), v.flatten(0, 1), [seq * i for i in range(batch + 1)], causal)
        assert torch.equal(packed.view_as(q), whole[0])
        ref = oracle.attention(*(t[:1].float().cpu().numpy() for t in (q, k, v)), causal)
        err = np.abs(whole[0][:1].float().cpu().numpy() - ref).max()
        assert err <= 2e-2 * max(1.0, np.abs(ref).max()), err


@pytest.mark.parametrize("head_dim", [72, 80, 88, 96])
@pytest.mark.parametrize("batch,n_q,n_kv,causal", [(1, 1, 1, True), (2, 33, 33, True), (1, 129, 129, True), (2, 40, 63, False), (3, 130, 65, False),
                                                   (4, 700, 520, False)])
def test_attention_heads_of_72_to_96(bd, head_dim, batch, n_q, n_kv, causal):
    """Heads that are padded to 80 and to 96, in workgroups of 4 wavefronts (12 pieces a row in LDS) and of 8 (the last): nothing but
    the head's own channels is read, as the rows lie in buffers of NaN, and every row is right.  Weights and output are rounded to
    bf16, 2^-9 each, the row sums are of the rounded weights: 2^-7 of the largest value covers them."""
    log("attention, heads of 72 to 96", head_dim, batch, n_q, n_kv, causal)
    g = torch.Generator(device="cuda").manual_seed(head_dim + n_q)

    def rows(n, heads):
        x = torch.full((batch, n, heads, head_dim + 8), float("nan"), dtype=torch.bfloat16, device="cuda")[..., :head_dim]
        return x.copy_(torch.randn(x.shape, generator=g, device="cuda"))

    q, k, v = rows(n_q, 16), rows(n_kv, 16), rows(n_kv, 16)
    out = bd.civic_prefill_attn(q, k, v, True) if causal else bd.civic_cross_attn(q, k, v)
    if batch == 4:
        assert bd.lib.civic_attn_workgroup(batch, n_q, n_kv, 16, 16, head_dim, 0) == 8
    qq, kk, vv = (x.double().transpose(1, 2).contiguous() for x in (q, k, v))
    z = torch.matmul(qq, kk.transpose(2, 3).contiguous()) / head_dim ** 0.5
    if causal:
        z.masked_fill_(torch.ones(n_q, n_kv, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    ref = torch.matmul(torch.softmax(z, -1), vv).transpose(1, 2)
    assert (out.double() - ref).abs().max().item() <= 2.0 ** -7 * ref.abs().max().item()


ITEM_ORDER = [
    # rows of the items, keys (0: the item's own), query and KV heads, head dim, causal, whether the items are shifted
    ((700, 20, 33, 25, 20, 10, 30, 21), 0, 16, 4, 64, True, True), ((640, 33, 1, 5), 0, 32, 4, 128, True, True),
    ((1200, 1, 1, 40), 0, 16, 8, 72, False, True), ((33, 900, 1, 257, 64, 31, 90, 140), 64, 16, 16, 80, False, True),
    ((520, 257, 1), 0, 16, 4, 128, True, False), ((300, 1, 290, 40, 161), 0, 8, 2, 96, True, False), ((700, 85, 300), 128, 12, 12, 64, False, False)]


@pytest.mark.parametrize("case", ITEM_ORDER)
def test_ragged_attention_order_of_items(bd, case):
    """Every row tile of every item once, in either order of the items (their shift by row tile also wraps around): the bits of a call
    for each item alone, and the items' rows in the caches."""
    rows, keys, q_heads, kv_heads, d, causal, _ = case
    log("ragged order", *case)
    g = torch.Generator(device="cuda").manual_seed(sum(rows) + d)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    kv_shape = (len(rows), keys, kv_heads, d) if keys else (int(off[-1]), kv_heads, d)
    q = torch.randn((int(off[-1]), q_heads, d), generator=g, device="cuda").bfloat16()
    k, v = (torch.randn(kv_shape, generator=g, device="cuda").bfloat16() for _ in range(2))
    out = torch.full_like(q, float("nan"))
    if keys:
        bd.civic_cross_attn_ragged(q, k, v, off, out=out)
        alone = [bd.civic_cross_attn(q[a:b][None], k[i:i + 1], v[i:i + 1])[0] for i, (a, b) in enumerate(zip(off[:-1], off[1:]))]
    else:
        kc, vc = (torch.full((len(rows), kv_heads, max(rows) + 3, d), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(2))
        bd.civic_prefill_attn_ragged(q, k, v, off, causal, 0.0, kc, vc, 2, out=out)
        alone = [bd.civic_prefill_attn(q[a:b][None], k[a:b][None], v[a:b][None], causal)[0] for a, b in zip(off[:-1], off[1:])]
        for i, (a, b) in enumerate(zip(off[:-1], off[1:])):
            for cache, x in ((kc, k), (vc, v)):
                assert torch.equal(cache[i, :, 2:2 + rows[i]], x[a:b].transpose(0, 1)) and cache[i, :, 2 + rows[i]:].isnan().all()
    assert torch.equal(out, torch.cat(alone))

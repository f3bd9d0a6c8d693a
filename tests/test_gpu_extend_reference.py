"""Rows whose score scale jumps after their first key tile (needs an MI355X).

The extend kernel takes a row's softmax reference from its first 64-key tile and raises it
only when a later tile outgrows it.  Here single keys of later tiles are
scaled so that the scores jump by hundreds (base 2), up and down, in some rows of a wave and
not in others: in unmasked tiles, on the diagonal, in the first and later chunks of a
split-KV call, and through the fused append.  A softmax over such scores is close to one-hot
and its error is that of bf16 weights and outputs, so the library's usual bounds hold.
"""
import numpy as np
import pytest
import torch

import paper_2608_10402_amd as tide
from gpu_harness import assert_close, assert_lse, host_f64, log

pytestmark = pytest.mark.gpu


def check_plan(kv, p, e, split):
    """TIDE_EXTEND_SPLIT cuts a call only where a block spans enough tiles: that it did."""
    info = tide.tide_plan_info_get(tide.TIDE_OP_EXTEND, np.array([p], np.int32),
                                   np.array([e], np.int32), kv.dims)
    assert info["split"] == int(split)


def build(hq, hkv, d, prefix, extend, scaled, seed, bad=None):
    """One task; keys `scaled` = {position: factor}; `bad` = (position, value) sets a key."""
    g = torch.Generator().manual_seed(seed)
    n = prefix + extend
    q = torch.randn((extend, hq, d), generator=g).bfloat16()
    k = torch.randn((n, hkv, d), generator=g)
    for pos, f in scaled.items():
        k[pos] *= f
    if bad:
        k[bad[0]] = bad[1]
    k = k.bfloat16()
    v = torch.randn((n, hkv, d), generator=g).bfloat16()
    x = torch.einsum("tghd,pgd->tghp", q.double().view(extend, hkv, hq // hkv, d), k.double()) / d ** 0.5
    seen = torch.arange(n) <= torch.arange(prefix, n)[:, None]
    x = x.masked_fill(~seen[:, None, None, :], -np.inf)
    w = torch.softmax(x, -1)
    ref = torch.einsum("tghp,pgd->tghd", w, v.double()).reshape(extend, hq, d).numpy()
    lse = torch.logsumexp(x, -1).reshape(extend, hq).numpy()
    pages = -(-n // 16)
    bt = np.random.default_rng(seed).permutation(pages).astype(np.int32).reshape(1, -1)
    kv = tide.PagedKV(pages, hq, hkv, d, bt)
    kv.append(k[:prefix].cuda(), v[:prefix].cuda(), [0], [prefix])
    return kv, q.cuda(), k[prefix:].cuda(), v[prefix:].cuda(), ref, lse


CASES = {
    "unmasked_jump": (4, 1, 128, 300, 40, {130: 64.0}),
    "two_jumps": (8, 2, 64, 500, 70, {70: 40.0, 333: 300.0}),
    "diagonal_jump": (7, 1, 128, 320, 100, {350: 200.0}),
    "first_tile_largest": (4, 2, 128, 260, 33, {5: 300.0}),
    "last_key": (2, 2, 64, 447, 1, {447: 500.0}),
    "long_split": (4, 2, 128, 2600, 50, {40: 30.0, 1000: 100.0, 2610: 400.0}),
}


@pytest.mark.parametrize("split", ["0", "1"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_score_jumps(name, split, monkeypatch):
    monkeypatch.setenv("TIDE_EXTEND_SPLIT", split)
    hq, hkv, d, p, e, scaled = CASES[name]
    log("jump case %s split %s" % (name, split))
    kv, q, kn, vn, ref, ref_lse = build(hq, hkv, d, p, e, scaled, seed=len(name))
    check_plan(kv, p, e, split)
    lse = torch.empty((e, hq), dtype=torch.float32, device="cuda")
    fused = kv.extend_append(q, kn, vn, [p], [e], lse=lse)
    assert_close(fused, ref, "%s fused" % name)
    # an fp32 log-sum-exp of magnitude 1e3 is good to about 1e-4 relative to its size
    tol = 1e-3 + 1e-6 * float(np.abs(ref_lse).max())
    assert_lse(lse, ref_lse, "%s fused" % name, tol)
    assert torch.equal(kv.extend(q, [p], [e]), fused)


@pytest.mark.parametrize("split", ["0", "1"])
@pytest.mark.parametrize("d", [64, 128])
def test_large_values_stay_finite(d, split, monkeypatch):
    """V of about 2^106 over rows whose scores jump by 0 to 60 (base 2) after their first tile.
    The weights a row keeps are below 2^8, so its sums stay below 2^121; the outputs are V's
    size, and their error relative to it is the usual one."""
    monkeypatch.setenv("TIDE_EXTEND_SPLIT", split)
    p, e = 400, 60
    log("large values d %d split %s" % (d, split))
    kv, q, kn, vn, ref, _ = build(8, 2, d, p, e, {150: 12.0, 333: 16.0}, seed=d)
    check_plan(kv, p, e, split)
    kv.v_pool.mul_(2.0 ** 106)
    out = kv.extend_append(q, kn, vn * 2.0 ** 106, [p], [e])
    assert_close(out.double() * 2.0 ** -106, ref, "large values")


@pytest.mark.parametrize("split", ["0", "1"])
def test_rows_do_not_depend_on_their_wave(split, monkeypatch):
    """A wave takes tiles' maxima before or after their weights, as its rows need.  Rows whose
    references are raised in many tiles, and rows whose are never, give the same bits whatever
    the rows between them are."""
    monkeypatch.setenv("TIDE_EXTEND_SPLIT", split)
    p, e = 2000, 64
    scaled = {70 + 61 * i: 4.0 + i for i in range(30)}  # growing outliers
    kv, q, kn, vn, ref, _ = build(4, 1, 128, p, e, scaled, seed=11)
    check_plan(kv, p, e, split)
    out = kv.extend_append(q, kn, vn, [p], [e])
    assert_close(out, ref, "growing outliers")
    for calm in (slice(0, None, 2), slice(1, None, 2), slice(0, None, 7)):
        other = q.clone()
        other[calm] *= 0.01  # their scores stay within the slack
        got = kv.extend(other, [p], [e])
        rest = torch.ones(e, dtype=torch.bool, device="cuda")
        rest[calm] = False
        assert torch.equal(got[rest], out[rest])
        alone = kv.extend((q * 0.01).bfloat16(), [p], [e])
        assert torch.equal(got[calm], alone[calm])


@pytest.mark.parametrize("lse", [False, True])
def test_dominant_weight_is_exact(lse):
    """Two keys of a later tile that outgrow the first by 10 to 40 (base 2), nearly equal, with
    opposite V.  The larger is the row's reference, so its weight is exactly 1 and only the
    other's is rounded to bf16; were both rounded, the error would be 1.4 times as large.  The
    bound is the error of that arithmetic in 64 bits over the same rows (about 1,000, each
    with an independent rounding: 5% of noise), times 1.15."""
    hq, hkv, d, p, e = 8, 1, 128, 250, 600
    g = torch.Generator().manual_seed(5)
    q = torch.randn((e, hq, d), generator=g).bfloat16()
    k = torch.randn((p + e, hkv, d), generator=g)
    v = torch.randn((p + e, hkv, d), generator=g).bfloat16()
    a, b = 130, 157
    k[a] *= 12
    k[b] = k[a] + 0.1 * torch.randn((hkv, d), generator=g)
    k = k.bfloat16()
    v[a], v[b] = 1.0, -1.0
    bt = np.random.default_rng(1).permutation(-(-(p + e) // 16)).astype(np.int32).reshape(1, -1)
    kv = tide.PagedKV(bt.size, hq, hkv, d, bt)
    kv.append(k[:p].cuda(), v[:p].cuda(), [0], [p])
    buf = torch.empty((e, hq), dtype=torch.float32, device="cuda") if lse else None
    out = kv.extend_append(q.cuda(), k[p:].cuda(), v[p:].cuda(), [p], [e], lse=buf)

    x = q.double().view(e * hq, d) @ k.double().view(-1, d).t() / d ** 0.5 * np.log2(np.e)
    seen = torch.arange(p + e) <= torch.arange(p, p + e).repeat_interleave(hq)[:, None]
    x = x.masked_fill(~seen, -np.inf)
    top = x[:, [a, b]].min(1).values - x[:, :64].max(1).values
    rows = (top > 10) & (top < 40) & (x.argmax(1) // 64 == a // 64)
    x = x[rows] - x[rows].max(1, keepdim=True).values
    w = torch.exp2(x)
    vd = v.double().view(-1, d)
    ref = w @ vd / w.sum(1, keepdim=True)
    w = w.bfloat16().double()
    model = (w @ vd / w.sum(1, keepdim=True)).bfloat16().double()
    got = out.double().cpu().view(e * hq, d)[rows]
    err, bound = (((t - ref) ** 2).mean().sqrt().item() for t in (got, model))
    log("dominant weight: %d rows, rms error %.3e, of the exact reference %.3e" % (rows.sum(), err, bound))
    assert rows.sum() > 800 and err <= 1.15 * bound


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_bad_key_stays_in_its_rows(value):
    """A key that holds NaN (or infinities, whose scores are infinite or NaN) reaches exactly
    the rows that see it."""
    p, e, at = 300, 40, 320
    log("bad key %s" % value)
    kv, q, kn, vn, _, _ = build(4, 1, 128, p, e, {}, seed=3, bad=(at, value))
    good = build(4, 1, 128, p, e, {}, seed=3)
    out = host_f64(kv.extend_append(q, kn, vn, [p], [e]))
    ref = host_f64(good[0].extend_append(*good[1:4], [p], [e]))
    assert np.array_equal(out[: at - p], ref[: at - p])
    assert np.isnan(out[at - p:]).any(axis=-1).any(axis=-1).all()

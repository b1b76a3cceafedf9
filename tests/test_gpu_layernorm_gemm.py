"""Transformer blocks whose LayerNorms go into the linear layers behind them (rows normalised on the way into the matrix cores), against the oracle and, to the
bit, against a launch for every norm: small launches of either type, ragged rows, the larger tiles, which get the norm as a launch of its own."""
import numpy as np
import pytest
import torch

import synthetic_inputs as SI
from configs import CONFIGS
from gpu_util import DEV, dev, dev_bytes, dev_f32, host, nchw_to_nhwc, nhwc_to_nchw, p, quantize, rel_l2, stream_ptr, tdtype
from oracle.unet import UNetConfig, weight_manifest
from paper_2406_06911_amd import binding as B
from test_gpu_pipeline import Case

pytestmark = pytest.mark.gpu

BF, F32 = B.AD_BF16, B.AD_F32
AUTO, REGISTERS, D2_128, P3_128, P3_256, P3_64, W4_256, D2_160, D2_320, K2_64 = -1, 3, 4, 5, 6, 7, 10, 14, 15, 16


def config(c, depth, height, width, batch, frames=0):
    return dict(latent_channels=4, height=height, width=width, batch=batch, channels=[c], layers_per_block=1, transformer_depth=[depth], mid_depth=0,
                head_dim=64, gn_groups=8, ctx_len=77, ctx_dim=64, pooled_dim=0, frames=frames, temporal_heads=4 if frames else 0)


def block(monkeypatch, d, dtype, tile, wts, spoil=None):
    """What the transformer of the first level adds to a stored input, the same of the oracle, the names of the launches."""
    monkeypatch.setitem(CONFIGS, "norms", d)
    B.check(B.lib.ad_tune_conv_tile(tile))
    try:
        case = Case("norms", dtype, 3, 1, 1, 1, cuts=[2, 3], wts=wts)
        trace = []
        case.oracle.run(case.noise, case.text, case.pooled, trace=trace)
        before, after = trace[0][1][1], trace[1][1][2]
        x = dev(nchw_to_nhwc(before), dtype)
        if spoil:
            spoil(x)
        out = [case.alloc_unit(u) for u in case.m.component_io(2)[1]]
        case.m.profile(True)
        case.m.component_forward(2, [x if u == 1 else None for u in case.m.component_io(2)[0]], 0, case.d_text, out, torch.cuda.current_stream())
        torch.cuda.synchronize()
        names = [r[0] for r in case.m.profile_records()]
        return nhwc_to_nchw(host(out[case.m.component_io(2)[1].index(2)]) - host(x)), after - before, names
    finally:
        B.check(B.lib.ad_tune_conv_tile(-1))


def by_launches(d, dtype, wts, x):
    """The same block (no frames) from the single-kernel entry points, a launch for every norm; x on the GPU, [batch][h][w][c]."""
    n, h, w, c = x.shape
    m, l, lk, lp, lkp = n * h * w, h * w, d["ctx_len"], (h * w + 63) // 64 * 64, (d["ctx_len"] + 63) // 64 * 64
    vt = dtype == BF                          # transposed values: the MFMA attention kernels
    empty = lambda *shape: torch.zeros(shape, device=DEV, dtype=tdtype(dtype))

    def linear(src, rows, cin, names, bias=None, residual=None, mode=B.OUT_ROWMAJOR, batch=1, ld_t=0):
        wt = np.concatenate([wts[t] for t in names])
        n_out = wt.shape[0]
        wp = dev_bytes(B.pack_conv_weight(dtype, wt.reshape(n_out, cin, 1, 1), mode == B.OUT_GEGLU))
        b = None
        if bias:
            b = np.zeros((n_out + 127) // 128 * 128, np.float32)
            r = np.arange(n_out)
            b[:n_out] = wts[bias][np.where(r % 64 < 32, r // 64 * 32 + r % 64, n_out // 2 + r // 64 * 32 + r % 64 - 32) if mode == B.OUT_GEGLU else r]
            b = dev_f32(b)
        third = empty(batch, n_out // 3, ld_t) if ld_t and mode == B.OUT_QKV else empty(rows, c)
        out = [empty(batch, n_out, ld_t) if mode == B.OUT_TRANSPOSED else empty(rows, {B.OUT_QKV: c, B.OUT_GEGLU: n_out // 2}.get(mode, n_out)), empty(rows, c), third]
        ws = B.lib.ad_conv_workspace_bytes(dtype, batch, rows // batch, 1, n_out, cin, 1, mode)
        scratch = torch.zeros(max(ws, 16), dtype=torch.uint8, device=DEV)
        B.check(B.lib.ad_conv_forward(dtype, p(src), None, cin, 0, batch, rows // batch, 1, 0, 1, 1, p(wp), n_out, p(b), None, p(residual), p(out[0]), p(out[1]), p(out[2]),
                                      mode, ld_t, p(scratch) if ws else None, ws, stream_ptr()))
        torch.cuda.synchronize()
        return out if mode == B.OUT_QKV else out[0]

    def norm(src, name):
        out, g, b = empty(m, c), dev_f32(wts[name + ".g"]), dev_f32(wts[name + ".b"])
        B.check(B.lib.ad_layernorm_forward(dtype, p(src), m, c, p(g), p(b), 1e-5, p(out), stream_ptr()))
        torch.cuda.synchronize()
        return out

    def attention(q, k, v, keys, ld_v):
        out = empty(m, c)
        B.check(B.lib.ad_attention_forward(dtype, p(q), p(k), p(v), int(vt), n, l, keys, c, d["head_dim"], c, c, ld_v if vt else c, c, p(out), stream_ptr()))
        torch.cuda.synchronize()
        return out

    t, text = "d0.0.tfm.", dev(quantize(SI.make_text(n, lk, d["ctx_dim"]), dtype), dtype)
    y, g, b = empty(m, c), dev_f32(wts[t + "gn.g"]), dev_f32(wts[t + "gn.b"])
    scratch = torch.zeros(B.lib.ad_groupnorm_scratch_bytes(n, l, c) // 4 + 4, device=DEV)
    B.check(B.lib.ad_groupnorm_forward(dtype, p(x), None, c, 0, n, l, d["gn_groups"], p(g), p(b), 1e-5, 0, p(y), p(scratch), stream_ptr()))
    rows = linear(y, m, c, [t + "proj_in.w"], t + "proj_in.b")
    for k in range(d["transformer_depth"][0]):
        s = "%s%d." % (t, k)
        q, key, v = linear(norm(rows, s + "ln1"), m, c, [s + "attn1.%s.w" % i for i in "qkv"], mode=B.OUT_QKV, batch=n, ld_t=lp if vt else 0)
        rows = linear(attention(q, key, v, l, lp), m, c, [s + "attn1.o.w"], s + "attn1.o.b", rows)
        q = linear(norm(rows, s + "ln2"), m, c, [s + "attn2.q.w"])
        key = linear(text, n * lk, d["ctx_dim"], [s + "attn2.k.w"])
        v = linear(text, n * lk, d["ctx_dim"], [s + "attn2.v.w"], mode=B.OUT_TRANSPOSED if vt else B.OUT_ROWMAJOR, batch=n, ld_t=lkp if vt else 0)
        rows = linear(attention(q, key, v, lk, lkp), m, c, [s + "attn2.o.w"], s + "attn2.o.b", rows)
        inner = linear(norm(rows, s + "ln3"), m, c, [s + "ff1.w"], s + "ff1.b", mode=B.OUT_GEGLU)
        rows = linear(inner, m, 4 * c, [s + "ff2.w"], s + "ff2.b", rows)
    return linear(rows, m, c, [t + "proj_out.w"], t + "proj_out.b", x)


def one_norm(d, row, spread, site, scale, rng):
    """Weights with which the tokens enter as `row` (and N(0, spread)) and the block is that plus `scale` times the layers behind one norm: site 1 the
    self-attention, 3 the feed-forward."""
    wts = SI.make_weights(weight_manifest(UNetConfig(**d)), std=d["channels"][0] ** -0.5, bf16_exact=True)
    t, c = "d0.0.tfm.", d["channels"][0]
    for name in wts:
        if name.startswith(t) and ".ln" in name:
            wts[name] = (rng.standard_normal(c) * 0.3 + name.endswith(".g")).astype(np.float32)
    last = {1: "0.attn1.o.w", 3: "0.ff2.w"}[site]
    for name in ["proj_out.b"] + ["0.%s.%s" % (o, v) for o in ("attn1.o", "attn2.o", "ff2") for v in "wb"]:
        wts[t + name] *= np.float32(scale if name == last else 0)
    wts[t + "proj_in.w"] *= np.float32(spread)
    wts[t + "proj_in.b"] = (row + np.zeros(c)).astype(np.float32)
    wts[t + "proj_out.w"] = np.eye(c, dtype=np.float32)
    return wts


@pytest.mark.parametrize("dtype,tile,c,depth,height,width,batch,frames,separate", [(BF, *p) for p in [
    (AUTO, 192, 2, 4, 4, 1, 0, False), (AUTO, 256, 2, 5, 3, 2, 0, False), (AUTO, 256, 1, 3, 5, 5, 5, False), (AUTO, 192, 1, 12, 12, 2, 0, False), (AUTO, 1280, 1, 3, 3, 1, 0, False),
    (AUTO, 192, 1, 33, 35, 2, 0, True), (AUTO, 320, 1, 61, 59, 1, 0, True),
    (AUTO, 640, 1, 13, 11, 1, 0, True), (AUTO, 320, 1, 48, 46, 3, 3, True),
    (D2_128, 320, 1, 13, 11, 2, 0, True), (P3_128, 256, 2, 13, 11, 2, 0, True), (P3_256, 320, 1, 23, 13, 2, 0, True), (P3_64, 192, 2, 13, 11, 2, 0, True),
    (D2_160, 320, 1, 13, 11, 3, 3, True), (D2_320, 320, 2, 23, 13, 2, 0, True), (D2_320, 448, 1, 9, 7, 1, 0, True), (K2_64, 192, 2, 13, 11, 2, 0, True), (K2_64, 320, 1, 3, 5, 5, 5, True),
    (REGISTERS, 192, 1, 13, 11, 2, 0, True), (W4_256, 256, 1, 13, 11, 2, 0, True)]] + [(F32, *p) for p in [
    (AUTO, 128, 1, 12, 12, 2, 0, False), (AUTO, 128, 2, 5, 3, 1, 0, False), (AUTO, 192, 1, 3, 5, 5, 5, False), (AUTO, 256, 2, 6, 6, 2, 0, False), (AUTO, 192, 1, 12, 12, 2, 0, False), (AUTO, 320, 1, 3, 3, 1, 0, False),
    (REGISTERS, 128, 1, 6, 6, 2, 0, True), (AUTO, 256, 1, 48, 46, 2, 0, True)]])
def test_layernorm_inside_the_linear_layer_matches_oracle(monkeypatch, dtype, tile, c, depth, height, width, batch, frames, separate):
    d = config(c, depth, height, width, batch, frames)
    wts = SI.make_weights(weight_manifest(UNetConfig(**d)), std=c ** -0.5, bf16_exact=dtype == BF)
    rng = np.random.default_rng(5)
    for name in wts:                          # gains and offsets that show when they are lost or land on other channels
        if ".ln" in name:
            wts[name] = (rng.standard_normal(wts[name].shape) * 0.3 + name.endswith(".g")).astype(np.float32)
    got, want, names = block(monkeypatch, d, dtype, tile, wts)
    # what the block adds: some ten roundings of 1.1e-3 on the way (input, hidden rows, norms, q, probabilities, inner rows, result), were they all to add up
    # (measured 5.5e-3 to 7.7e-3); fp32: ten sums of a few hundred terms, 1.5e-7 each (measured 3.1e-7 to 6.7e-7)
    err = rel_l2(got, want)
    assert np.isfinite(got).all() and err < (1.1e-2 if dtype == BF else 1.5e-6), err
    assert (names.count("layernorm") > 0) == separate, names


# edges of the sums of a row: fewer accesses of 16 bytes than lanes (24, 32), 64 and more, no multiple of 64 (72, 80, 160), row tiles of 16 and 32, rows beyond the tensor
@pytest.mark.parametrize("dtype,c,depth,height,width,batch", [(BF, *q) for q in [
    (192, 2, 4, 4, 1), (256, 2, 5, 3, 2), (192, 1, 12, 12, 2), (320, 1, 9, 5, 1), (576, 1, 5, 4, 2), (640, 1, 9, 5, 1), (1280, 1, 3, 3, 1), (1280, 1, 10, 9, 2)]] + [
    (F32, *q) for q in [(128, 1, 12, 12, 2), (192, 1, 12, 12, 2), (256, 2, 6, 6, 2), (320, 1, 3, 3, 1), (640, 1, 3, 3, 1)]])
def test_same_bits_as_a_launch_for_every_norm(monkeypatch, dtype, c, depth, height, width, batch):
    d = config(c, depth, height, width, batch)
    wts = SI.make_weights(weight_manifest(UNetConfig(**d)), std=c ** -0.5, bf16_exact=dtype == BF)
    rng = np.random.default_rng(17)
    for name in wts:
        if ".ln" in name:
            wts[name] = (rng.standard_normal(wts[name].shape) * 0.3 + name.endswith(".g")).astype(np.float32)
    kept = []
    got, _, names = block(monkeypatch, d, dtype, AUTO, wts, spoil=kept.append)
    x = kept[0]
    want = nhwc_to_nchw(host(by_launches(d, dtype, wts, x).reshape(x.shape)) - host(x))
    assert "layernorm" not in names or (dtype, c, batch) == (BF, 1280, 2), names       # there two of the three layers have too much of K for a small tile
    assert np.isfinite(got).all() and np.array_equal(got, want), rel_l2(got, want)


@pytest.mark.parametrize("site", [1, 3])
@pytest.mark.parametrize("c,offset,spread", [(128, 10, 1), (256, 10, 1), (128, 100, 1), (256, 100, 1), (320, 100, 1), (256, 1000, 1), (256, 77.1, 0)])
def test_fp32_rows_with_an_offset(monkeypatch, c, offset, spread, site):
    """Rows whose mean is 10 to 1000 standard deviations, and rows of one value, which the norm turns into its own offset: nothing is lost of them that a launch
    for every norm keeps."""
    d, kept = config(c, 1, 5, 4, 2), []
    wts = one_norm(d, offset, spread, site, 2.0 ** 14, np.random.default_rng(7))
    got, _, names = block(monkeypatch, d, F32, AUTO, wts, spoil=kept.append)
    x = kept[0]
    want = nhwc_to_nchw(host(by_launches(d, F32, wts, x).reshape(x.shape)) - host(x))
    assert "layernorm" not in names and np.abs(want).max() > 1 and np.array_equal(got, want), (names, rel_l2(got, want))


@pytest.mark.parametrize("dtype", [F32, BF])
@pytest.mark.parametrize("value,finite", [(1e30, True), (float("inf"), False)])
def test_rows_with_a_huge_value(monkeypatch, dtype, value, finite):
    """1e30 in a channel: its square is beyond the type, the norm leaves its offset.  Infinity: no number in any row.  Both as with a launch for every norm."""
    d, kept = config(192, 1, 5, 4, 2), []
    row = np.zeros(192)
    row[100] = value
    wts = one_norm(d, row, 1, 1, 1, np.random.default_rng(19))
    with np.errstate(all="ignore"):
        got, _, names = block(monkeypatch, d, dtype, AUTO, wts, spoil=kept.append)
    x = kept[0]
    want = nhwc_to_nchw(host(by_launches(d, dtype, wts, x).reshape(x.shape)) - host(x))
    assert "layernorm" not in names and np.isfinite(got).all() == finite and np.array_equal(got, want, equal_nan=True)


@pytest.mark.parametrize("dtype,c", [(F32, 128), (F32, 256), (BF, 192), (BF, 256)])
def test_a_sample_of_nan_stays_by_itself(monkeypatch, dtype, c):
    """Samples of 15 rows share row tiles: one that is not a number comes out as such, and the other to the same bits as without it."""
    d = config(c, 1, 5, 3, 2)
    wts = SI.make_weights(weight_manifest(UNetConfig(**d)), std=c ** -0.5, bf16_exact=True)
    clean, _, names = block(monkeypatch, d, dtype, AUTO, wts)
    got, _, _ = block(monkeypatch, d, dtype, AUTO, wts, spoil=lambda x: x[1].fill_(float("nan")))
    assert "layernorm" not in names and np.isfinite(clean).all()
    assert (got[0] == clean[0]).all() and np.isnan(got[1]).all()


@pytest.mark.parametrize("tile,c", [(AUTO, 192), (AUTO, 256), (AUTO, 320), (P3_64, 256), (P3_128, 256), (D2_320, 320)])
def test_gains_are_not_rounded_into_the_weights(monkeypatch, tile, c):
    """Rows of +-32, gains of any value and offsets that bring the norm's result to +-1, whole weights whose products cancel down to 1 .. 3: every number
    that is stored in 16 bits is exact, gain x weight would not be."""
    d, rng = config(c, 1, 5, 4, 2), np.random.default_rng(11)
    sign = rng.permutation(np.repeat([1.0, -1.0], c // 2))
    wts = one_norm(d, 32 * sign, 0, 1, 1, rng)
    t = "d0.0.tfm.0."
    wts[t + "ln1.b"] = (sign * (1 - wts[t + "ln1.g"].astype(np.float64))).astype(np.float32)
    v = rng.integers(-4, 5, (c, c))
    for r in range(c):                        # each row's sum over the signs becomes 1, 2 or 3
        while (gap := r % 3 + 1 - int(v[r] @ sign)) != 0:
            k = rng.integers(c)
            if abs(v[r, k] + np.sign(gap) * sign[k]) <= 8:
                v[r, k] += int(np.sign(gap) * sign[k])
    wts[t + "attn1.v.w"] = v.astype(np.float32)
    wts[t + "attn1.o.w"] = 64 * np.eye(c, dtype=np.float32)
    got, want, names = block(monkeypatch, d, BF, tile, wts)
    assert ("layernorm" in names) == (tile != AUTO), names
    # three roundings of at most 2^-9 (the block's input and output, the probabilities' sum)
    assert rel_l2(got, want) < 6e-3, rel_l2(got, want)


@pytest.mark.parametrize("site", [1, 3])
@pytest.mark.parametrize("tile,c,count", [(AUTO, 192, 11), (AUTO, 320, 13), (AUTO, 576, 11), (P3_64, 320, 13)])
def test_bf16_rows_with_an_offset(monkeypatch, tile, c, count, site):
    """Rows of 772 and a few 776, neighbours in bf16: a mean of 800 standard deviations or more.  The variance has to come from the deviations: the mean of
    the squares less the square of the mean is off by 2 to 7 % of the deviation here, in fp32, where the mean is no short binary fraction."""
    d, rng = config(c, 1, 5, 4, 2), np.random.default_rng(13)
    row = np.full(c, 772.0)
    row[rng.permutation(c)[:count]] = 776
    got, want, names = block(monkeypatch, d, BF, tile, one_norm(d, row, 0, site, 2.0 ** 14, rng))
    assert ("layernorm" in names) == (tile != AUTO), names
    # seven roundings of 1.1e-3 (norm, value or inner row, probabilities, hidden row, result) and a mean off by two of its own, 9e-5 of a standard deviation
    assert rel_l2(got, want) < 8e-3, rel_l2(got, want)

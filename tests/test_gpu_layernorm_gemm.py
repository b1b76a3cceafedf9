"""Transformer blocks whose LayerNorms go into the linear layers behind them (rows normalised on the way into the matrix cores, sums of the rows from the
launch in front), against the oracle: small launches of either type, ragged rows, the larger tiles, which get the norm as a launch of its own."""
import numpy as np
import pytest
import torch

import synthetic_inputs as SI
from configs import CONFIGS
from gpu_util import dev, host, nchw_to_nhwc, nhwc_to_nchw, rel_l2
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


@pytest.mark.parametrize("site", [1, 3])
@pytest.mark.parametrize("c,offset,spread", [(128, 10, 1), (256, 10, 1), (128, 100, 1), (256, 100, 1), (320, 100, 1), (256, 1000, 1), (256, 77.1, 0)])
def test_fp32_rows_with_an_offset(monkeypatch, c, offset, spread, site):
    """Rows whose mean is 10 to 1000 standard deviations, and rows of one value, which the norm turns into its own offset: the norm inside the linear layer
    loses no more of them than as a launch of its own (which the register-staged kernels have in front of them)."""
    d = config(c, 1, 5, 4, 2)
    wts = one_norm(d, offset, spread, site, 2.0 ** 14, np.random.default_rng(7))
    got, want, names = block(monkeypatch, d, F32, AUTO, wts)
    apart, _, names_apart = block(monkeypatch, d, F32, REGISTERS, wts)
    assert "layernorm" not in names and names_apart.count("layernorm") == 3, (names, names_apart)
    # half as much again for the luck of other roundings of the mean; 3e-7: the sums behind the norm
    err, err_apart = rel_l2(got, want), rel_l2(apart, want)
    assert err < 1.5 * err_apart + 3e-7, (err, err_apart)


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

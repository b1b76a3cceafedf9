"""Transformer blocks whose LayerNorms go into the linear layers behind them (gains in the weights, offsets in the bias, sums of the rows from the launch in
front), against the oracle: every tile that takes part, ragged rows, the kernels that do not and get the norm as a launch of its own."""
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


@pytest.mark.parametrize("dtype,tile,c,depth,height,width,batch,frames,separate", [(BF, *p) for p in [
    (AUTO, 192, 2, 4, 4, 1, 0, False), (AUTO, 256, 2, 5, 3, 2, 0, False), (AUTO, 256, 1, 3, 5, 5, 5, False), (AUTO, 192, 1, 33, 35, 2, 0, False), (AUTO, 320, 1, 61, 59, 1, 0, False),
    (AUTO, 640, 1, 13, 11, 1, 0, False), (AUTO, 320, 1, 48, 46, 3, 3, False),
    (D2_128, 320, 1, 13, 11, 2, 0, False), (P3_128, 256, 2, 13, 11, 2, 0, False), (P3_256, 320, 1, 23, 13, 2, 0, False), (P3_64, 192, 2, 13, 11, 2, 0, False),
    (D2_160, 320, 1, 13, 11, 3, 3, False), (D2_320, 320, 2, 23, 13, 2, 0, False), (D2_320, 448, 1, 9, 7, 1, 0, False), (K2_64, 192, 2, 13, 11, 2, 0, False), (K2_64, 320, 1, 3, 5, 5, 5, False),
    (REGISTERS, 192, 1, 13, 11, 2, 0, True), (W4_256, 256, 1, 13, 11, 2, 0, True)]] + [(F32, *p) for p in [
    (AUTO, 128, 1, 12, 12, 2, 0, False), (AUTO, 128, 2, 5, 3, 1, 0, False), (AUTO, 192, 1, 3, 5, 5, 5, False), (AUTO, 256, 2, 6, 6, 2, 0, False), (AUTO, 320, 1, 3, 3, 1, 0, False),
    (REGISTERS, 128, 1, 6, 6, 2, 0, True), (AUTO, 256, 1, 48, 46, 2, 0, True)]])
def test_layernorm_inside_the_linear_layer_matches_oracle(monkeypatch, dtype, tile, c, depth, height, width, batch, frames, separate):
    d = dict(latent_channels=4, height=height, width=width, batch=batch, channels=[c], layers_per_block=1, transformer_depth=[depth], mid_depth=0,
             head_dim=64, gn_groups=8, ctx_len=77, ctx_dim=64, pooled_dim=0, frames=frames, temporal_heads=4 if frames else 0)
    monkeypatch.setitem(CONFIGS, "norms", d)
    wts = SI.make_weights(weight_manifest(UNetConfig(**d)), std=c ** -0.5, bf16_exact=dtype == BF)
    rng = np.random.default_rng(5)
    for name in wts:                          # gains and offsets that show when they are lost or land on other channels
        if ".ln" in name:
            wts[name] = (rng.standard_normal(wts[name].shape) * 0.3 + name.endswith(".g")).astype(np.float32)
    B.check(B.lib.ad_tune_conv_tile(tile))
    try:
        case = Case("norms", dtype, 3, 1, 1, 1, cuts=[2, 3], wts=wts)
        trace = []
        case.oracle.run(case.noise, case.text, case.pooled, trace=trace)
        before, after = trace[0][1][1], trace[1][1][2]
        x = dev(nchw_to_nhwc(before), dtype)
        out = [case.alloc_unit(u) for u in case.m.component_io(2)[1]]
        case.m.profile(True)
        case.m.component_forward(2, [x if u == 1 else None for u in case.m.component_io(2)[0]], 0, case.d_text, out, torch.cuda.current_stream())
        torch.cuda.synchronize()
        names = [r[0] for r in case.m.profile_records()]
        got = nhwc_to_nchw(host(out[case.m.component_io(2)[1].index(2)]) - host(x))
        # what the block adds: some ten roundings of 1.1e-3 on the way (input, hidden rows, weights behind a norm, q, probabilities, inner rows, result) and the
        # sums behind them, 4-8e-3 in all; fp32: sums of a few hundred terms, 1e-6
        err = rel_l2(got, after - before)
        assert np.isfinite(got).all() and err < (2e-2 if dtype == BF else 1e-5), err
        assert (names.count("layernorm") > 0) == separate, names
    finally:
        B.check(B.lib.ad_tune_conv_tile(-1))

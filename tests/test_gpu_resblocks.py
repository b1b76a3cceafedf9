"""ResBlocks against the oracle, one at a time: the shortcut as further k-tiles of the second convolution (every LDS-DMA tile, K-splits that begin
behind the taps, one and two sources, ragged rows and columns)."""
import numpy as np
import pytest
import torch

import synthetic_inputs as SI
from configs import CONFIGS
from gpu_util import DEV, dev, dev_bytes, dev_f32, host, nchw_to_nhwc, nhwc_to_nchw, p, rel_l2, stream_ptr, tdtype
from paper_2406_06911_amd import binding as B
from test_gpu_pipeline import Case

pytestmark = pytest.mark.gpu


def check_blocks(monkeypatch, dtype, tile, channels, height, width, batch, wanted, groups=8):
    d = dict(latent_channels=4, height=height, width=width, batch=batch, channels=channels, layers_per_block=1, transformer_depth=[0, 0], mid_depth=0,
             head_dim=64, gn_groups=groups, ctx_len=8, ctx_dim=64, pooled_dim=0)
    monkeypatch.setitem(CONFIGS, "blocks", d)
    B.check(B.lib.ad_tune_conv_tile(tile))
    try:
        probe = B.AsyncDiff(d, 1, 0, 1, dtype)
        units = probe.units()
        probe.close()
        blocks = [i for i, u in enumerate(units) if ".res" in u.name.decode() and wanted(u)]
        assert blocks
        for i in blocks:
            case = Case("blocks", dtype, 3, 1, 1, 1, std=(9 * channels[0]) ** -0.5, cuts=[i, i + 1])
            trace = []
            case.oracle.run(case.noise, case.text, case.pooled, trace=trace)
            stored = trace[0][1]
            ins, outs = case.m.component_io(2)
            out = [case.alloc_unit(u) for u in outs]
            case.m.component_forward(2, [dev(nchw_to_nhwc(stored[u]), dtype) for u in ins], 0, case.d_text, out, torch.cuda.current_stream())
            torch.cuda.synchronize()
            ref, got = trace[1][1][i], nhwc_to_nchw(host(out[outs.index(i)]))
            # bf16: five roundings on the way (inputs, both normalised tensors, the first convolution, the result), 1.1e-3 each: 2.5e-3 in all, five
            # times that for a single element; fp32: sums of a few thousand terms.  One k-tile too many or too few is a few percent at least.
            rel, most = (5e-3, 0.025) if dtype == B.AD_BF16 else (1e-5, 1e-4)
            assert rel_l2(got, ref) < rel, (units[i].name, rel_l2(got, ref))
            assert np.all(np.abs(got - ref) < most * (np.sqrt(np.mean(ref ** 2)) + np.abs(ref))), units[i].name
    finally:
        B.check(B.lib.ad_tune_conv_tile(-1))


@pytest.mark.parametrize("tile,channels,height,width,batch", [
    (4, [128, 192], 22, 14, 2), (5, [128, 192], 22, 14, 2), (6, [128, 192], 22, 14, 2), (7, [128, 192], 22, 14, 2), (14, [128, 192], 22, 14, 2), (16, [128, 192], 22, 14, 2), (16, [64, 320], 34, 18, 2), (16, [128, 192], 6, 4, 1),
    (15, [128, 192], 22, 14, 2), (5, [64, 64], 2, 2, 1), (7, [64, 320], 34, 18, 2), (-1, [320, 640], 20, 18, 1), (-1, [64, 320], 72, 40, 1),
    (-1, [320, 320], 48, 46, 2)])
def test_shortcut_inside_the_second_convolution(monkeypatch, tile, channels, height, width, batch):
    check_blocks(monkeypatch, B.AD_BF16, tile, channels, height, width, batch, lambda u: u.c_in + u.c_skip != u.c_out)


@pytest.mark.parametrize("dtype,tile,channels,height,width,batch", [
    (B.AD_BF16, t, [128, 192], 22, 14, 2) for t in (1, 3, 8, 9, 10, 11, 12)] + [
    (B.AD_F32, t, [64, 96], 22, 14, 1) for t in (1, 3, -1)] + [
    (B.AD_BF16, -1, [64, 128], 8, 6, 1), (B.AD_BF16, 15, [64, 448], 12, 10, 1), (B.AD_F32, -1, [32, 64], 6, 4, 1)])
def test_weights_in_blocks_in_every_kernel(monkeypatch, dtype, tile, channels, height, width, batch):
    """The kernel families that the test above leaves out read a model's weights in blocks of 32 rows; tiles that end beyond the padded rows."""
    check_blocks(monkeypatch, dtype, tile, channels, height, width, batch, lambda u: True)


def from_single_kernels(d, dtype, wts, name, x0, x1, c_out):
    """A ResBlock from the single-kernel entry points, a launch for every norm and for the shortcut (whose sum passes through the storage type)."""
    n, h, w, c0 = x0.shape
    c1 = 0 if x1 is None else x1.shape[3]

    def norm(a, b, part):
        c = a.shape[3] + (0 if b is None else b.shape[3])
        out, g, o = torch.empty(n, h, w, c, device=DEV, dtype=tdtype(dtype)), dev_f32(wts[name + part + ".g"]), dev_f32(wts[name + part + ".b"])
        scratch = torch.zeros(B.lib.ad_groupnorm_scratch_bytes(n, h * w, c) // 4 + 4, device=DEV)
        B.check(B.lib.ad_groupnorm_forward(dtype, p(a), p(b), a.shape[3], c - a.shape[3], n, h * w, d["gn_groups"], p(g), p(o), 1e-5, 1, p(out), p(scratch), stream_ptr()))
        torch.cuda.synchronize()
        return out

    def conv(a, b, part, k, rowvec=None, residual=None):
        wt = wts[name + part + ".w"]
        wp, bias = dev_bytes(B.pack_conv_weight(dtype, wt)), np.zeros((c_out + 127) // 128 * 128, np.float32)
        bias[:c_out] = wts[name + part + ".b"]
        bias, out = dev_f32(bias), torch.empty(n, h, w, c_out, device=DEV, dtype=tdtype(dtype))
        cb = 0 if b is None else b.shape[3]
        ws = B.lib.ad_conv_workspace_bytes(dtype, n, h, w, c_out, a.shape[3] + cb, k, B.OUT_ROWMAJOR)
        scratch = torch.zeros(max(ws, 16), dtype=torch.uint8, device=DEV)
        B.check(B.lib.ad_conv_forward(dtype, p(a), p(b), a.shape[3], cb, n, h, w, 0, k, 1, p(wp), c_out, p(bias), p(rowvec), p(residual), p(out), None, None, B.OUT_ROWMAJOR, 0,
                                      p(scratch) if ws else None, ws, stream_ptr()))
        torch.cuda.synchronize()
        return out

    rowvec = dev_f32(np.tile(wts[name + "temb.b"], (n, 1)))           # the time projection's weights are 0
    y = norm(conv(norm(x0, x1, "gn1"), None, "conv1", 3, rowvec), None, "gn2")
    short = x0 if c0 + c1 == c_out else conv(x0, x1, "short", 1)
    return conv(y, None, "conv2", 3, residual=short)


# tiles of 16x16, 16x32 and 32x32; the shortcut's k-tiles fewer than, as many as and more than the wavefronts, beginning with each of them; one and two sources
@pytest.mark.parametrize("dtype,channels,groups,height,width,batch", [
    (B.AD_BF16, [128, 256], 32, 6, 6, 2), (B.AD_BF16, [64, 128], 32, 24, 24, 2), (B.AD_BF16, [256, 256], 32, 6, 6, 2), (B.AD_BF16, [64, 128], 8, 34, 18, 1), (B.AD_BF16, [192, 128], 32, 6, 6, 2),
    (B.AD_BF16, [64, 64], 32, 48, 46, 2), (B.AD_BF16, [64, 256], 32, 32, 32, 2), (B.AD_F32, [32, 64], 8, 16, 16, 1), (B.AD_F32, [64, 128], 32, 24, 24, 2), (B.AD_F32, [128, 256], 32, 12, 12, 2),
    (B.AD_F32, [256, 256], 32, 6, 6, 2), (B.AD_F32, [96, 32], 8, 10, 6, 2), (B.AD_F32, [32, 64], 8, 34, 30, 1)])
def test_small_tiles_have_the_bits_of_separate_launches(dtype, channels, groups, height, width, batch):
    d = dict(latent_channels=4, height=height, width=width, batch=batch, channels=channels, layers_per_block=1, transformer_depth=[0, 0], mid_depth=0,
             head_dim=64, gn_groups=groups, ctx_len=8, ctx_dim=64, pooled_dim=0)
    probe = B.AsyncDiff(d, 1, 0, 1, dtype)
    units = probe.units()
    wts = SI.make_weights(probe.weight_manifest(), std=(9 * channels[0]) ** -0.5, bf16_exact=dtype == B.AD_BF16)
    probe.close()
    rng = np.random.default_rng(41)
    for name in wts:
        if ".gn" in name:
            wts[name] = (rng.standard_normal(wts[name].shape) * 0.3 + name.endswith(".g")).astype(np.float32)
        if name.endswith("temb.w"):
            wts[name] *= np.float32(0)
    small = 0
    for i, u in enumerate(units):
        if ".res" not in u.name.decode():
            continue
        m = B.AsyncDiff(d, 3, 1, 1, dtype, cuts=[i, i + 1])
        m.allocate(DEV)
        m.load_weights(wts)
        m.reset(2)
        ins, outs = m.component_io(2)
        text = torch.zeros(batch, 8, 64, device=DEV, dtype=tdtype(dtype))
        store = {v: dev(rng.standard_normal(m.tensor_shape(v)[0]), dtype) for v in ins}
        out = {v: torch.full(m.tensor_shape(v)[0], float("nan"), device=DEV, dtype=tdtype(dtype)) for v in outs}
        m.profile(True)
        m.component_forward(2, [store[v] for v in ins], 0, text, [out[v] for v in outs], torch.cuda.current_stream())
        torch.cuda.synchronize()
        names = [r[0] for r in m.profile_records() if not r[0].startswith(("time", "linear_rows"))]
        m.close()
        if any("igemm" in n and not n.endswith("small") for n in names):       # other tiles keep the shortcut's sum in fp32
            continue
        small += 1
        want = from_single_kernels(d, dtype, wts, u.name.decode() + ".", store[i - 1], store[u.skip_from] if u.c_skip else None, u.c_out)
        assert torch.equal(out[i], want), (u.name, rel_l2(host(out[i]), host(want)), names)
    assert small >= 2

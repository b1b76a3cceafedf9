"""ResBlocks against the oracle, one at a time: the shortcut as further k-tiles of the second convolution (every LDS-DMA tile, K-splits that begin
behind the taps, one and two sources, ragged rows and columns)."""
import numpy as np
import pytest
import torch

from configs import CONFIGS
from gpu_util import dev, host, nchw_to_nhwc, nhwc_to_nchw, rel_l2
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

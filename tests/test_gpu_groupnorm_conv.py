"""GroupNorm inside the 3x3 convolution behind it (small maps): the output head against 64 bits on inputs of all kinds, ResBlocks against the oracle.  Tiles that
begin and end in the middle of samples and image rows, one and two sources, a group in a quarter of an access to four of them, both types."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

from gpu_util import DEV, dev, quantize, rel_l2
from paper_2406_06911_amd import binding as B
from test_gpu_resblocks import check_blocks

pytestmark = pytest.mark.gpu


def config(channels, height, width, batch, groups):
    return dict(latent_channels=4, height=height, width=width, batch=batch, channels=channels, layers_per_block=1, transformer_depth=[0] * len(channels), mid_depth=0,
                head_dim=64, gn_groups=groups, ctx_len=8, ctx_dim=64, pooled_dim=0)


def head(d, dtype, x, gain, offset, w, bias):
    """The output head alone (second component of two) on x [batch][h][w][c]; result, names of the launches of the component."""
    probe = B.AsyncDiff(d, 1, 0, 1, dtype)
    last = len(probe.units()) - 1
    probe.close()
    m = B.AsyncDiff(d, 2, 1, 1, dtype, cuts=[last])
    m.allocate(DEV)
    mine = {"out.gn.g": gain, "out.gn.b": offset, "out.conv.w": w, "out.conv.b": bias}
    m.load_weights({n: mine.get(n, np.zeros(s, np.float32)) for n, s in m.weight_manifest()})
    m.reset(2)
    text = torch.zeros(d["batch"], d["ctx_len"], d["ctx_dim"], device=DEV, dtype=x.dtype)
    out = torch.full((d["batch"], 4, d["height"], d["width"]), float("nan"), device=DEV)
    m.profile(True)
    m.component_forward(2, [x], 0, text, [out], torch.cuda.current_stream())
    torch.cuda.synchronize()
    names = [r[0] for r in m.profile_records()]
    m.profile(False)
    m.close()
    return out.cpu().numpy().astype(np.float64), names


SHAPES = [  # dtype, channels, height, width, batch, groups, in one launch
    (B.AD_BF16, 256, 3, 3, 2, 32, True), (B.AD_BF16, 256, 6, 6, 2, 32, True), (B.AD_BF16, 128, 12, 12, 2, 32, True), (B.AD_BF16, 64, 10, 14, 1, 32, True),
    (B.AD_BF16, 64, 16, 20, 1, 8, True), (B.AD_BF16, 64, 17, 19, 1, 8, False), (B.AD_BF16, 512, 2, 4, 2, 16, False), (B.AD_BF16, 128, 1, 1, 1, 8, True),
    (B.AD_BF16, 192, 6, 6, 2, 32, False), (B.AD_BF16, 128, 5, 7, 2, 64, True), (B.AD_BF16, 64, 24, 24, 2, 32, False),
    (B.AD_F32, 32, 16, 16, 1, 8, True), (B.AD_F32, 64, 12, 12, 2, 32, True), (B.AD_F32, 128, 12, 12, 2, 32, True), (B.AD_F32, 256, 6, 6, 2, 32, True), (B.AD_F32, 512, 3, 3, 1, 32, True), (B.AD_F32, 1024, 2, 2, 1, 64, False),
    (B.AD_F32, 128, 5, 7, 1, 64, True), (B.AD_F32, 32, 3, 7, 2, 8, True), (B.AD_F32, 96, 6, 6, 1, 8, False)]


@pytest.mark.parametrize("kind", ["plain", "offset", "outlier", "constant"])
@pytest.mark.parametrize("dtype,c,height,width,batch,groups,fused", SHAPES)
def test_head(dtype, c, height, width, batch, groups, fused, kind):
    d = config([c], height, width, batch, groups)
    rng = np.random.default_rng(c + height)
    x = rng.standard_normal((batch, height, width, c)).astype(np.float32)
    if kind == "offset":
        x += 100.0 * rng.standard_normal(c).astype(np.float32)[None, None, None, :]
    if kind == "outlier":
        x[:, -1, -1, ::3] = 30.0
    if kind == "constant":
        x[-1] = 7.0                                                   # a sample without variance: eps alone
    x = quantize(x, dtype)
    gain, offset = (1 + 0.3 * rng.standard_normal(c)).astype(np.float32), (0.3 * rng.standard_normal(c)).astype(np.float32)
    w, bias = quantize(rng.standard_normal((4, c, 3, 3)) * (9 * c) ** -0.5, dtype), rng.standard_normal(4).astype(np.float32)
    got, names = head(d, dtype, dev(x, dtype), gain, offset, w, bias)
    assert ("gn_group" not in names and "gn_apply" not in names) == fused, names
    t = torch.from_numpy(x).double().permute(0, 3, 1, 2)
    y = F.silu(F.group_norm(t, groups, torch.from_numpy(gain).double(), torch.from_numpy(offset).double(), 1e-5))
    if dtype == B.AD_BF16:
        y = y.float().bfloat16().double()                             # the operand of the matrix cores
    ref = F.conv2d(y, torch.from_numpy(np.asarray(w)).double(), torch.from_numpy(bias).double(), padding=1).numpy()
    # fp32: sums of 9 c terms and a dozen roundings on the way, 6e-8 each.  bf16: the same operands but for the few that fp32 rounds to the other neighbour
    # (1e-6 of a value moves one in some thousand by 2^-8, less than 2e-4 in all)
    assert rel_l2(got, ref) < (5e-4 if dtype == B.AD_BF16 else 3e-6), rel_l2(got, ref)
    assert np.abs(got - ref).max() < (1e-2 if dtype == B.AD_BF16 else 3e-5) * np.sqrt(np.mean(ref ** 2))


@pytest.mark.parametrize("dtype,channels,height,width,batch,groups", [
    (B.AD_BF16, [256, 256], 6, 6, 2, 32), (B.AD_BF16, [128, 128], 12, 12, 2, 32), (B.AD_BF16, [64, 64], 4, 12, 2, 8), (B.AD_F32, [32, 32], 12, 4, 1, 8),
    (B.AD_F32, [64, 64], 6, 10, 2, 16), (B.AD_BF16, [64, 64], 24, 26, 2, 32), (B.AD_F32, [128, 256], 6, 6, 2, 32), (B.AD_BF16, [64, 256], 2, 2, 1, 32), (B.AD_BF16, [192, 128], 6, 6, 2, 32)])
def test_blocks(monkeypatch, dtype, channels, height, width, batch, groups):
    """Two sources, the time projection of each sample, residuals, shortcuts."""
    check_blocks(monkeypatch, dtype, -1, channels, height, width, batch, lambda u: True, groups)


@pytest.mark.parametrize("dtype,channels,height,width,batch,groups,launches", [
    (B.AD_BF16, [128, 256], 6, 6, 2, 32, 2), (B.AD_F32, [64, 128], 6, 6, 2, 32, 2),              # both norms and the shortcut inside the convolutions
    (B.AD_BF16, [64, 128], 48, 48, 2, 32, 4), (B.AD_BF16, [192, 128], 6, 6, 2, 32, 3)])          # the norms of larger maps, and of 192 channels, are launches
def test_launches_of_a_block_that_changes_its_width(dtype, channels, height, width, batch, groups, launches):
    d = config(channels, height, width, batch, groups)
    probe = B.AsyncDiff(d, 1, 0, 1, dtype)
    units = [u.name.decode() for u in probe.units()]
    probe.close()
    i = units.index("d1.0.res")                                       # channels[0] -> channels[1] on a quarter of the pixels
    m = B.AsyncDiff(d, 3, 1, 1, dtype, cuts=[i, i + 1])
    m.allocate(DEV)
    m.load_weights({n: np.full(s, 0.01, np.float32) for n, s in m.weight_manifest()})
    m.reset(2)
    ins, outs = m.component_io(2)
    store = {}
    for u in ins + outs:
        b, h, w, c = m.tensor_shape(u)[0]
        store[u] = torch.ones(b, h, w, c, device=DEV, dtype=torch.bfloat16 if dtype == B.AD_BF16 else torch.float32)
    text = torch.zeros(batch, 8, 64, device=DEV, dtype=store[ins[0]].dtype)
    m.profile(True)
    m.component_forward(2, [store[u] for u in ins], 0, text, [store[u] for u in outs], torch.cuda.current_stream())
    torch.cuda.synchronize()
    names = [r[0] for r in m.profile_records() if not r[0].startswith(("time", "linear_rows"))]
    m.close()
    assert len(names) == launches, names


@pytest.mark.parametrize("dtype,channels,height,width", [(B.AD_BF16, [128, 64], 6, 6), (B.AD_F32, [64, 32], 6, 6), (B.AD_BF16, [64, 128], 12, 12)])
def test_a_block_whose_result_overwrites_its_input(dtype, channels, height, width):
    """hidden_out may be hidden_in: the launches that would read what others have overwritten are then the separate ones."""
    d = config(channels, 2 * height, 2 * width, 1, 8)
    probe = B.AsyncDiff(d, 1, 0, 1, dtype)
    units = [u.name.decode() for u in probe.units()]
    probe.close()
    i = units.index("d1.0.res")
    m = B.AsyncDiff(d, 3, 1, 1, dtype, cuts=[i, i + 1])
    m.allocate(DEV)
    rng = np.random.default_rng(3)
    m.load_weights({n: (rng.standard_normal(s) * 0.05 + (len(s) == 1 and n.endswith(".g"))).astype(np.float32) for n, s in m.weight_manifest()})
    m.reset(2)
    (u_in,), (u_out,) = [[u for u in us if u in (i - 1, i)] for us in m.component_io(2)]
    shape_in, shape_out = m.tensor_shape(u_in)[0], m.tensor_shape(u_out)[0]
    t = torch.bfloat16 if dtype == B.AD_BF16 else torch.float32
    x = torch.from_numpy(rng.standard_normal(shape_in[0] * shape_in[1] * shape_in[2] * shape_in[3]).astype(np.float32)).to(DEV).to(t)
    size = shape_out[0] * shape_out[1] * shape_out[2] * shape_out[3]
    text = torch.zeros(1, 8, 64, device=DEV, dtype=t)

    def run(src, dst):
        ins, outs = m.component_io(2)
        m.component_forward(2, [src if u == u_in else None for u in ins], 0, text, [dst if u == u_out else None for u in outs], torch.cuda.current_stream())
        torch.cuda.synchronize()
        return dst[:size].float().cpu()

    apart = run(x.clone(), torch.empty(max(size, x.numel()), device=DEV, dtype=t))
    both = torch.empty(max(size, x.numel()), device=DEV, dtype=t)
    both[:x.numel()] = x
    same = run(both, both)
    m.close()
    # the shortcut's sum passes through the storage type in the separate launches: one rounding (2^-9 of a value) and what follows from it
    assert rel_l2(same.numpy(), apart.numpy()) < (4e-3 if dtype == B.AD_BF16 else 1e-6)


@pytest.mark.parametrize("dtype", [B.AD_BF16, B.AD_F32])
def test_an_input_between_two_accesses(dtype):
    """hidden_in 8 bytes behind a multiple of 16: the norm is a launch of its own."""
    c, size = 64, 12
    d = config([c], size, size, 2, 32)
    rng = np.random.default_rng(4)
    x = quantize(rng.standard_normal((2, size, size, c)), dtype)
    gain, offset = (1 + 0.3 * rng.standard_normal(c)).astype(np.float32), (0.3 * rng.standard_normal(c)).astype(np.float32)
    w, bias = quantize(rng.standard_normal((4, c, 3, 3)) * (9 * c) ** -0.5, dtype), rng.standard_normal(4).astype(np.float32)
    at16 = dev(x, dtype)
    skip = 8 // at16.element_size()
    moved = torch.empty(at16.numel() + 16, device=DEV, dtype=at16.dtype)[skip:skip + at16.numel()].view(at16.shape)
    moved.copy_(at16)
    want, _ = head(d, dtype, at16, gain, offset, w, bias)
    got, names = head(d, dtype, moved, gain, offset, w, bias)
    assert any(n.startswith("gn_") for n in names), names
    # other order of the sums of the statistics: fp32 roundings, and the few bf16 operands that these move
    assert rel_l2(got, want) < (5e-4 if dtype == B.AD_BF16 else 3e-6)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("dtype,c,size", [(B.AD_BF16, 256, 3), (B.AD_F32, 64, 6)])
def test_a_sample_that_is_not_finite(dtype, c, size, value):
    """Rows of both samples meet in a tile: the finite one keeps its bits, the other has no value anywhere, as with a launch for the norm."""
    d = config([c], size, size, 2, 32)
    rng = np.random.default_rng(6)
    x = quantize(rng.standard_normal((2, size, size, c)), dtype)
    gain, offset = np.ones(c, np.float32), np.zeros(c, np.float32)
    w, bias = quantize(rng.standard_normal((4, c, 3, 3)) * (9 * c) ** -0.5, dtype), np.zeros(4, np.float32)
    want, names = head(d, dtype, dev(x, dtype), gain, offset, w, bias)
    assert not any(n.startswith("gn_") for n in names), names
    for z in range(2):
        broken = x.copy()
        broken[z, size // 2, size // 2, 5] = value
        got, _ = head(d, dtype, dev(broken, dtype), gain, offset, w, bias)
        assert np.array_equal(got[1 - z], want[1 - z])
        assert np.isnan(got[z]).all()

"""GroupNorm inside the 3x3 convolution behind it (small maps): the output head against 64 bits on inputs of all kinds, ResBlocks against the oracle.  Tiles that
begin and end in the middle of samples and image rows, one and two sources, a group in a quarter of an access to four of them, both types."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

from gpu_util import DEV, dev, dev_bytes, dev_f32, p, quantize, rel_l2, stream_ptr
from paper_2406_06911_amd import binding as B
from test_gpu_resblocks import check_blocks

pytestmark = pytest.mark.gpu


def config(channels, height, width, batch, groups):
    return dict(latent_channels=4, height=height, width=width, batch=batch, channels=channels, layers_per_block=1, transformer_depth=[0] * len(channels), mid_depth=0,
                head_dim=64, gn_groups=groups, ctx_len=8, ctx_dim=64, pooled_dim=0, frames=batch if batch > 2 else 0, temporal_heads=8 if batch > 2 else 0)


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
    # one rounding of the shortcut's sum to the storage type (2^-9 of a value) and what follows from it; the small tiles round it as the separate launches do
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
    # fp32 roundings, and the few bf16 operands that these move, were the sums of the statistics taken in another order
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


def by_launches(d, dtype, x, gain, offset, w, bias):
    """The head from the single-kernel entry points, a launch for the norm."""
    n, h, wd, c = x.shape
    y = torch.empty_like(x)
    scratch = torch.zeros(B.lib.ad_groupnorm_scratch_bytes(n, h * wd, c) // 4 + 4, device=DEV)
    g, o, b = dev_f32(gain), dev_f32(offset), dev_f32(np.concatenate([bias, np.zeros(124, np.float32)]))
    B.check(B.lib.ad_groupnorm_forward(dtype, p(x), None, c, 0, n, h * wd, d["gn_groups"], p(g), p(o), 1e-5, 1, p(y), p(scratch), stream_ptr()))
    wp, out = dev_bytes(B.pack_conv_weight(dtype, w)), torch.full((n, 4, h, wd), float("nan"), device=DEV)
    B.check(B.lib.ad_conv_forward(dtype, p(y), None, c, 0, n, h, wd, 0, 3, 1, p(wp), 4, p(b), None, None, p(out), None, None, B.OUT_TRANSPOSED_F32, h * wd, None, 0, stream_ptr()))
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


def on_a_boundary(rng, shape, groups, mean):
    """Groups whose mean is a number of few bits: sums of it that differ in their last bit are cut off to different 12 bits."""
    n, h, w, c = shape
    x = rng.standard_normal((n, h * w, groups, c // groups))
    return (x - x.mean(axis=(1, 3), keepdims=True) + mean).reshape(shape).astype(np.float32)


# every arrangement of samples in the lanes: one sample, two, three; sizes of a power of two side by side; more than 256 accesses of a group (16x20, 24x24, 17x18)
SAME_BITS = [s[:6] for s in SHAPES if s[6]] + [
    (B.AD_BF16, 64, 16, 16, 1, 32), (B.AD_BF16, 128, 8, 8, 2, 32), (B.AD_BF16, 256, 3, 3, 4, 32), (B.AD_BF16, 256, 2, 2, 16, 32), (B.AD_BF16, 256, 1, 1, 16, 32), (B.AD_BF16, 128, 2, 4, 5, 32),
    (B.AD_BF16, 256, 5, 8, 2, 32), (B.AD_BF16, 256, 4, 4, 3, 8), (B.AD_BF16, 256, 6, 6, 2, 16), (B.AD_BF16, 128, 12, 13, 1, 8), (B.AD_BF16, 256, 6, 6, 1, 64),
    (B.AD_F32, 32, 24, 24, 1, 8), (B.AD_F32, 64, 17, 18, 1, 8), (B.AD_F32, 32, 17, 17, 2, 8), (B.AD_F32, 64, 8, 8, 2, 16), (B.AD_F32, 256, 3, 3, 3, 32), (B.AD_F32, 256, 2, 1, 8, 32), (B.AD_F32, 128, 6, 7, 2, 8),
    (B.AD_F32, 256, 6, 6, 2, 64), (B.AD_F32, 32, 1, 1, 7, 8)]


@pytest.mark.parametrize("kind", ["plain", "boundary", "offset", "huge"])
@pytest.mark.parametrize("dtype,c,height,width,batch,groups", SAME_BITS)
def test_same_bits_as_a_launch_for_the_norm(dtype, c, height, width, batch, groups, kind):
    d = config([c], height, width, batch, groups)
    rng = np.random.default_rng(29 + c + height)
    shape = (batch, height, width, c)
    x = on_a_boundary(rng, shape, groups, 8.0) if kind == "boundary" else rng.standard_normal(shape)
    if kind == "offset":
        x = x + 100.0 * rng.standard_normal(c)
    if kind == "huge":
        x = 7e17 * x
    x = dev(quantize(x, dtype), dtype)
    gain, offset = (1 + 0.3 * rng.standard_normal(c)).astype(np.float32), (0.3 * rng.standard_normal(c)).astype(np.float32)
    w, bias = quantize(rng.standard_normal((4, c, 3, 3)) * (9 * c) ** -0.5, dtype), rng.standard_normal(4).astype(np.float32)
    got, names = head(d, dtype, x, gain, offset, w, bias)
    assert not any(n.startswith("gn_") for n in names), names
    want = by_launches(d, dtype, x, gain, offset, w, bias)
    assert np.isfinite(got).all() and np.array_equal(got, want), rel_l2(got, want)


def picked(d, dtype, x, gain, offset, channels):
    """The normalised values of four channels, as they are: the head's weights take a channel each, at the middle tap."""
    w = np.zeros((4, x.shape[3], 3, 3), np.float32)
    w[np.arange(4), channels, 1, 1] = 1
    got, names = head(d, dtype, dev(x, dtype), gain, offset, w, np.zeros(4, np.float32))
    assert not any(n.startswith("gn_") for n in names), names
    t = torch.from_numpy(x).double().permute(0, 3, 1, 2)
    ref = F.silu(F.group_norm(t, d["gn_groups"], torch.from_numpy(gain).double(), torch.from_numpy(offset).double(), 1e-5))
    return got, ref[:, list(channels)].numpy()


@pytest.mark.parametrize("mean", [1.0, 8.0, 100.0])
@pytest.mark.parametrize("c,size,groups", [(32, 16, 8), (64, 12, 8), (128, 12, 32)])
def test_fp32_means_on_a_boundary_of_twelve_bits(c, size, groups, mean):
    """Every lane has to take the same number off the values of a group before their squares are summed."""
    d, rng = config([c], size, size, 1, groups), np.random.default_rng(31)
    ones, zeros = np.ones(c, np.float32), np.zeros(c, np.float32)
    for i in range(8):
        x = on_a_boundary(rng, (1, size, size, c), groups, mean)
        channels = rng.permutation(groups)[:4] * (c // groups)
        got, ref = picked(d, B.AD_F32, x, ones, zeros, channels)
        # a value of up to 5: ten roundings, 6e-8 each; the mean of up to 1024 deviations, each exact but for one rounding
        assert np.abs(got - ref).max() < 5e-6, (i, np.abs(got - ref).max())


@pytest.mark.parametrize("dtype,c,size,groups", [(B.AD_F32, 32, 16, 8), (B.AD_BF16, 64, 16, 8)])
def test_squares_whose_sum_is_beyond_fp32(dtype, c, size, groups):
    """7e17 squared 1024 or 2048 times: beyond fp32 in all, not in a quarter of them.  The norm has a value, not its offset."""
    d, rng = config([c], size, size, 1, groups), np.random.default_rng(37)
    scale = 7e17 if dtype == B.AD_F32 else 5e17
    x = quantize(scale * rng.choice([-1.0, 1.0], (1, size, size, c)), dtype)
    ones, zeros = np.ones(c, np.float32), np.zeros(c, np.float32)
    got, ref = picked(d, dtype, x, ones, zeros, rng.permutation(groups)[:4] * (c // groups))
    # fp32: as above.  bf16: one rounding of the operand, 2^-9
    assert np.abs(got - ref).max() < (4e-3 if dtype == B.AD_BF16 else 5e-6), np.abs(got - ref).max()


def replay(x, gain, offset, per):
    """One group of one sample, x [pixels][channels] fp32, as k_gn_group adds it up: thread t of 256 takes the access of `per` channels t % vpp of pixels t // vpp, + 256 // vpp, ...,
    the first two squares fused as a0 a0 + (a1 a1), the lanes of a wavefront pairwise, the wavefronts in order, in double for the deviations."""
    f32, f64 = np.float32, np.float64
    hw, c = x.shape
    vpp = c // per
    fma = lambda a, b, z: (f64(a) * f64(b) + f64(z)).astype(f32)      # the product is exact in 64 bits
    rounds = -(-hw * vpp // 256)
    held = np.zeros((rounds * 256, per), f32)
    held[:hw * vpp] = x.reshape(hw * vpp, per)
    live = (np.arange(rounds * 256) < hw * vpp).reshape(rounds, 256)
    held = held.reshape(rounds, 256, per)

    def lanes(v):
        v = v.reshape(4, 64)
        while v.shape[1] > 1:
            v = v[:, ::2] + v[:, 1::2]
        return v[:, 0]

    s = np.zeros(256, f32)
    for r in range(rounds):
        for e in range(per):
            s = s + held[r, :, e]
    total = f32(0)
    for v in lanes(s):
        total = total + v
    about = (np.array([total * f32(1.0 / (hw * c))], f32).view(np.uint32) & np.uint32(0xfffff000)).view(f32)[0]
    s, q = np.zeros(256, f32), np.zeros(256, f32)
    for r in range(rounds):
        d = np.where(live[r][:, None], held[r] - about, f32(0))
        for e in range(per):
            s = s + d[:, e]
        q = fma(d[:, 0], d[:, 0], d[:, 1] * d[:, 1] if r == 0 else q)
        for e in range(2 if r == 0 else 1, per):
            q = fma(d[:, e], d[:, e], q)
    more = np.sum(lanes(s).astype(f64)) * (1.0 / (hw * c))
    var = np.sum(lanes(q).astype(f64)) * (1.0 / (hw * c)) - more * more + f64(f32(1e-5))
    ga = gain * f32(1 / np.sqrt(var))
    return fma(x - about, ga, fma(-f32(more), ga, offset))


@pytest.mark.parametrize("c,hw,groups", [(64, 36, 16), (64, 144, 32), (128, 300, 16), (32, 256, 8), (256, 90, 16)])
def test_order_of_the_sums_of_the_norm_by_itself(c, hw, groups):
    """The norm's own kernel keeps its bits: what is compared with it elsewhere would not show that it changed."""
    rng = np.random.default_rng(43)
    x = (rng.standard_normal((2, hw, c)) + 3).astype(np.float32)
    gain, offset = (1 + 0.3 * rng.standard_normal(c)).astype(np.float32), (0.3 * rng.standard_normal(c)).astype(np.float32)
    d, g, o = dev_f32(x), dev_f32(gain), dev_f32(offset)
    out, scratch = torch.empty_like(d), torch.zeros(B.lib.ad_groupnorm_scratch_bytes(2, hw, c) // 4 + 4, device=DEV)
    B.check(B.lib.ad_groupnorm_forward(B.AD_F32, p(d), None, c, 0, 2, hw, groups, p(g), p(o), 1e-5, 0, p(out), p(scratch), stream_ptr()))
    torch.cuda.synchronize()
    got, cpg = out.cpu().numpy(), c // groups
    differ = 0
    for z in range(2):
        for k in range(groups):
            at = slice(k * cpg, (k + 1) * cpg)
            differ += np.count_nonzero(replay(x[z][:, at], gain[at], offset[at], min(cpg, 4)) != got[z][:, at])
    # the replay rounds twice where a kernel's fused product rounds once (one in 2^29), and takes 1 / sqrt exactly; another order of the sums is 1 to 10 %
    assert differ <= 1e-3 * got.size, differ / got.size


@pytest.mark.parametrize("second", [False, True])
@pytest.mark.parametrize("dtype,channels,size,unit,small", [
    (B.AD_BF16, [64, 128], 12, "u1.1.res", True), (B.AD_BF16, [64, 64], 12, "u1.1.res", True), (B.AD_F32, [32, 64], 12, "u1.1.res", True), (B.AD_BF16, [64, 128], 24, "u0.1.res", True),
    (B.AD_BF16, [64, 128], 96, "u0.0.res", False)])
def test_a_block_of_two_sources_whose_result_overwrites_one(dtype, channels, size, unit, small, second):
    """hidden_out may be either input: the shortcut, which other workgroups would still read, is then a launch of its own."""
    d = config(channels, size, size, 1, 8)
    probe = B.AsyncDiff(d, 1, 0, 1, dtype)
    units = probe.units()
    probe.close()
    i = [u.name.decode() for u in units].index(unit)
    m = B.AsyncDiff(d, 3, 1, 1, dtype, cuts=[i, i + 1])
    m.allocate(DEV)
    rng = np.random.default_rng(47)
    m.load_weights({n: (rng.standard_normal(s) * 0.05 + (len(s) == 1 and n.endswith(".g"))).astype(np.float32) for n, s in m.weight_manifest()})
    m.reset(2)
    ins, outs = m.component_io(2)
    sources, t = [i - 1, units[i].skip_from], torch.bfloat16 if dtype == B.AD_BF16 else torch.float32
    assert set(sources) <= set(ins) and i in outs and units[i].c_skip
    shapes = {u: m.tensor_shape(u)[0] for u in sources + [i]}
    size_of = {u: int(np.prod(s)) for u, s in shapes.items()}
    x = {u: dev(rng.standard_normal(shapes[u]), dtype) for u in sources}
    text = torch.zeros(1, 8, 64, device=DEV, dtype=t)

    def run(out, at):
        m.profile(True)
        m.component_forward(2, [at.get(u) for u in ins], 0, text, [out if u == i else None for u in outs], torch.cuda.current_stream())
        torch.cuda.synchronize()
        names = [r[0] for r in m.profile_records() if r[0].startswith("igemm")]
        m.profile(False)
        return out[:size_of[i]].clone(), names

    apart, names = run(torch.empty(size_of[i], device=DEV, dtype=t), x)
    over = sources[second]
    both = torch.empty(max(size_of[i], size_of[over]), device=DEV, dtype=t)
    both[:size_of[over]] = x[over].flatten()
    same, more = run(both, {**x, over: both})
    m.close()
    assert len(names) == 2 and len(more) == 3, (names, more)          # both convolutions; and the shortcut
    assert all(n.endswith("small") for n in names) == small, names
    # the small tiles have the bits of a launch for the shortcut; the others round its sum once less (2^-9 of a value) and what follows from it
    assert torch.equal(same, apart) if small else rel_l2(same.float().cpu().numpy(), apart.float().cpu().numpy()) < 4e-3

"""The row-local transformer kernel of narrow models (k_tfm_rows) against the oracle's transformer block, at the sizes where it can go
wrong: token counts around its tiles of 16 and 32, key counts around its blocks, one and several layers, shared text, every head width."""
import ctypes as C

import numpy as np
import pytest
import torch

import synthetic_inputs as SI
from configs import CONFIGS
from gpu_util import DEV, assert_kernel_close, dev, dev_f32, host, nchw_to_nhwc, nhwc_to_nchw, p, quantize, rel_l2, stream_ptr
from oracle import primitives as P
from paper_2406_06911_amd import binding as B
from test_gpu_pipeline import Case, run_components_isolated

pytestmark = pytest.mark.gpu

BF, F32 = B.AD_BF16, B.AD_F32


@pytest.mark.parametrize("dtype,c,head_dim,depth,height,width,batch,ctx_len,frames", [
    (BF, 64, 64, 1, 4, 4, 1, 77, 0), (BF, 64, 64, 1, 5, 5, 2, 32, 0), (BF, 64, 64, 3, 17, 1, 2, 33, 0), (BF, 64, 64, 1, 65, 65, 2, 77, 0),
    (BF, 128, 64, 1, 3, 3, 1, 1, 0), (BF, 128, 64, 2, 13, 5, 2, 154, 0), (BF, 128, 64, 1, 8, 4, 5, 64, 5), (BF, 64, 64, 2, 3, 5, 3, 96, 3),
    (F32, 32, 16, 1, 4, 4, 1, 8, 0), (F32, 32, 32, 2, 5, 7, 2, 17, 0), (F32, 64, 16, 1, 1, 1, 1, 16, 0), (F32, 64, 32, 1, 11, 3, 3, 77, 3),
    (F32, 64, 64, 2, 9, 7, 2, 77, 0), (F32, 64, 16, 1, 91, 91, 1, 5, 0)])
def test_transformer_of_a_narrow_model_matches_oracle(monkeypatch, dtype, c, head_dim, depth, height, width, batch, ctx_len, frames):
    d = dict(latent_channels=4, height=height, width=width, batch=batch, channels=[c], layers_per_block=1, transformer_depth=[depth], mid_depth=0,
             head_dim=head_dim, gn_groups=8, ctx_len=ctx_len, ctx_dim=64, pooled_dim=0, frames=frames, temporal_heads=4 if frames else 0)
    monkeypatch.setitem(CONFIGS, "rows", d)
    # weights of about 1 / sqrt(width): the block adds as much as it is given
    case = Case("rows", dtype, 3, 1, 1, 1, std=c ** -0.5, cuts=[2, 3])
    assert [u.name.decode() for u in case.m.units()][2] == "d0.0.tfm"
    trace = []
    case.oracle.run(case.noise, case.text, case.pooled, trace=trace)
    before, after = trace[0][1][1], trace[1][1][2]
    x = dev(nchw_to_nhwc(before), dtype)
    out = [case.alloc_unit(u) for u in case.m.component_io(2)[1]]
    for _ in range(2):                       # the text's keys and values computed on the way, then from the cache
        case.m.component_forward(2, [x if u == 1 else None for u in case.m.component_io(2)[0]], 0, case.d_text, out, torch.cuda.current_stream())
        torch.cuda.synchronize()
        got = nhwc_to_nchw(host(out[case.m.component_io(2)[1].index(2)]) - host(x))
        # what the block adds.  bf16: some ten roundings of 1.1e-3 on the way (input, hidden rows, q, probabilities, inner rows, result) and
        # the sums behind them, 4-8e-3 in all; fp32: sums of a few hundred terms, 1e-6
        err = rel_l2(got, after - before)
        assert np.isfinite(got).all() and err < (2e-2 if dtype == BF else 1e-5), err
        case.m.precompute_text(case.d_text, torch.cuda.current_stream())


@pytest.mark.parametrize("dtype,c,frames,height,width,by_rows", [(BF, 128, 16, 32, 32, True), (BF, 128, 15, 33, 34, False), (BF, 64, 15, 33, 34, True), (F32, 64, 15, 33, 34, True)])
def test_transformer_of_many_tokens(monkeypatch, dtype, c, frames, height, width, by_rows):
    """Beyond 16384 tokens 128 bf16 channels go through the separate launches (their weights are packed for those): which way is taken, and the result."""
    names = []
    forward = B.AsyncDiff.component_forward

    def profiled(self, *args, **more):
        self.profile(True)
        forward(self, *args, **more)
        names.extend(r[0] for r in self.profile_records())

    monkeypatch.setattr(B.AsyncDiff, "component_forward", profiled)
    test_transformer_of_a_narrow_model_matches_oracle(monkeypatch, dtype, c, 64, 1, height, width, frames, 77, frames)
    assert any("tfm_rows" in n for n in names) == by_rows, set(names)


@pytest.mark.parametrize("dtype,c,batch,pooled,frames", [(F32, 32, 1, 0, 0), (F32, 64, 2, 8, 0), (BF, 64, 2, 128, 0), (BF, 64, 5, 0, 5), (BF, 128, 2, 16, 0),
                                                         (F32, 96, 1, 0, 0), (BF, 192, 2, 0, 0)])
def test_time_embedding_reaches_the_residual_blocks(monkeypatch, dtype, c, batch, pooled, frames):
    """Both ways of the time embedding: in one launch (up to 256 features in fp32, 362 in bf16, and few pooled ones) and layer by layer, with and without the
    pooled branch, at several timesteps (the ResBlock's output depends on them through the projection, whose weights are large here)."""
    d = dict(latent_channels=4, height=4, width=4, batch=batch, channels=[c], layers_per_block=1, transformer_depth=[0], mid_depth=0, head_dim=32,
             gn_groups=8, ctx_len=8, ctx_dim=64, pooled_dim=pooled, frames=frames, temporal_heads=4 if frames else 0)
    monkeypatch.setitem(CONFIGS, "temb", d)
    case = Case("temb", dtype, 2, 1, 1, 4, std=2 * c ** -0.5, cuts=[1])
    # 1e-4 / 2e-2: the budget of a component, asserted inside
    run_components_isolated(case)


@pytest.mark.parametrize("dtype,c,batch,pooled,fused", [(BF, 64, 1, 0, True), (BF, 64, 1, 384, True), (BF, 64, 1, 392, False), (BF, 64, 2, 224, True), (BF, 64, 2, 232, False),
                                                        (F32, 64, 1, 24, True), (F32, 64, 1, 32, False), (F32, 64, 2, 8, False), (F32, 32, 2, 592, True), (F32, 32, 2, 600, False)])
def test_time_embedding_in_one_launch_up_to_the_weights_a_workgroup_takes_in(monkeypatch, dtype, c, batch, pooled, fused):
    """The one launch reads the pooled branch's weights once a sample in every workgroup: around the line, which way is taken, and the result."""
    d = dict(latent_channels=4, height=4, width=4, batch=batch, channels=[c], layers_per_block=1, transformer_depth=[0], mid_depth=0, head_dim=32,
             gn_groups=8, ctx_len=8, ctx_dim=64, pooled_dim=pooled)
    monkeypatch.setitem(CONFIGS, "temb", d)
    # (the pooled branch's inputs grow with pooled_dim; weights that keep the embedding of unit size)
    case = Case("temb", dtype, 2, 1, 1, 2, std=(c + 4 * c + pooled) ** -0.5, cuts=[1])
    case.m.profile(True)
    run_components_isolated(case)
    names = {r[0] for r in case.m.profile_records()}
    assert ("time_fused" in names) == fused and ("linear_rows" in names) == (not fused), names


class StepRef(C.Structure):
    _fields_ = [("table", C.c_void_p), ("counter", C.c_void_p), ("offset", C.c_int)]


@pytest.mark.parametrize("dtype,dim,n", [(BF, 64, 1), (BF, 1024, 7), (BF, 1088, 6), (BF, 16384, 5), (BF, 16448, 5), (F32, 32, 3), (F32, 1056, 4), (F32, 33056, 9)])
def test_first_layer_of_the_time_embedding_at_any_width(dtype, dim, n):
    """The layer by itself (a whole model of the widest of these has gigabytes of weights): one and several pieces of the sinusoid, a short last one."""
    launch = getattr(B.lib, "_ZN2ad17launch_time_firstEifNS_7StepRefEiPKvPKfiPfP12ihipStream_t")       # ad::launch_time_first
    launch.argtypes = [C.c_int, C.c_float, StepRef, C.c_int, C.c_void_p, C.c_void_p, C.c_int, C.c_void_p, C.c_void_p]
    w, bias = quantize(SI.make_array((n, dim), 401, dim ** -0.5), dtype), SI.make_array((n,), 402)
    dw, db, out = dev(w, dtype), dev_f32(bias), torch.full((n,), float("nan"), device=DEV)
    for tau in (0, 999):
        B.check(launch(dtype, float(tau), StepRef(None, None, 0), dim, p(dw), p(db), n, p(out), stream_ptr()))
        torch.cuda.synchronize()
        assert_kernel_close(host(out), P.silu(P.linear(P.timestep_embedding(tau, dim), w, bias)), F32)

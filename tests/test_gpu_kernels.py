"""Kernel-level parity: every HIP kernel against the oracle's plain definition, through the C ABI."""
import ctypes as C
import math

import numpy as np
import pytest
import torch

import synthetic_inputs as SI
from gpu_util import (DEV, KTOL, TOL, assert_kernel_close, dev, dev_bytes, dev_f32, host, nchw_to_nhwc, nhwc_to_nchw, p, quantize, rel_l2, stream_ptr, tdtype)
from oracle import primitives as P
from oracle import sampler as SM
from paper_2406_06911_amd import binding as B

pytestmark = pytest.mark.gpu
lib = B.lib
DT = [B.AD_F32, B.AD_BF16]


def sync():
    torch.cuda.synchronize()


# ---------------------------------------------------------------------------------------------------
def run_conv(dtype, x0, x1, w, bias, stride=1, up=0, rowvec=None, residual=None, mode=B.OUT_ROWMAJOR, geglu=False, splitk=False):
    """x0/x1 NCHW float arrays (already quantised); returns the device result as float64 array."""
    n, c0, hs, ws = x0.shape
    c1 = x1.shape[1] if x1 is not None else 0
    k = w.shape[2]
    n_out = w.shape[0]
    d0 = dev(nchw_to_nhwc(x0), dtype)
    d1 = dev(nchw_to_nhwc(x1), dtype) if x1 is not None else None
    wp = dev_bytes(B.pack_conv_weight(dtype, w, geglu))
    nb = (n_out + 127) // 128 * 128
    bpad = np.zeros(nb, np.float32)
    if bias is not None:
        bb = np.asarray(bias, np.float32)
        if geglu:
            half = n_out // 2
            idx = [(r // 64) * 32 + r % 64 if r % 64 < 32 else half + (r // 64) * 32 + r % 64 - 32 for r in range(n_out)]
            bb = bb[idx]
        bpad[:n_out] = bb
    db = dev_f32(bpad) if bias is not None else None
    hin, win = hs << up, ws << up
    pad = k // 2
    ho, wo = (hin + 2 * pad - k) // stride + 1, (win + 2 * pad - k) // stride + 1
    drow = dev_f32(rowvec) if rowvec is not None else None
    dres = dev(residual, dtype) if residual is not None else None
    if mode == B.OUT_ROWMAJOR:
        out = torch.full((n, ho, wo, n_out), float("nan"), device=DEV, dtype=tdtype(dtype))
        ld_t = 0
    elif mode == B.OUT_GEGLU:
        out = torch.full((n, ho, wo, n_out // 2), float("nan"), device=DEV, dtype=tdtype(dtype))
        ld_t = 0
    else:
        ld_t = (ho * wo + 63) // 64 * 64
        out = torch.full((n, n_out, ld_t), float("nan"), device=DEV, dtype=tdtype(dtype) if mode == B.OUT_TRANSPOSED else torch.float32)
    ws_bytes = lib.ad_conv_workspace_bytes(dtype, n, ho, wo, n_out, c0 + c1, k, mode) if splitk else 0
    wsb = torch.zeros(max(ws_bytes, 16), dtype=torch.uint8, device=DEV)
    B.check(lib.ad_conv_forward(dtype, p(d0), p(d1), c0, c1, n, hs, ws, up, k, stride, p(wp), n_out, p(db), p(drow), p(dres),
                                p(out), None, None, mode, ld_t, p(wsb) if ws_bytes else None, ws_bytes, stream_ptr()))
    run_conv.last_ws_bytes = ws_bytes
    sync()
    return host(out), (ho, wo)


CONV_CASES = [
    # name, batch, c0, c1, hs, ws, n_out, k, stride, up
    ("3x3_multi_tile_ragged", 2, 64, 0, 13, 11, 192, 3, 1, 0),
    ("3x3_stride2", 2, 64, 0, 12, 10, 64, 3, 2, 0),
    ("3x3_upsampled", 1, 64, 0, 7, 9, 128, 3, 1, 1),
    ("3x3_concat", 2, 64, 128, 9, 9, 64, 3, 1, 0),
    ("1x1_concat", 2, 128, 64, 10, 9, 320, 1, 1, 0),
    ("3x3_small_n", 2, 64, 0, 8, 8, 4, 3, 1, 0),
    ("3x3_big_tiles", 2, 64, 0, 96, 96, 320, 3, 1, 0),
]


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("case", CONV_CASES, ids=[c[0] for c in CONV_CASES])
def test_conv_matches_direct_summation(dtype, case):
    name, n, c0, c1, hs, ws, n_out, k, stride, up = case
    x0 = quantize(SI.make_array((n, c0, hs, ws), 11), dtype)
    x1 = quantize(SI.make_array((n, c1, hs, ws), 12), dtype) if c1 else None
    w = quantize(SI.make_array((n_out, c0 + c1, k, k), 13, 0.05), dtype)
    bias = SI.make_array((n_out,), 14, 0.1)
    got, (ho, wo) = run_conv(dtype, x0, x1, w, bias, stride, up)
    xin = x0 if x1 is None else np.concatenate([x0, x1], 1)
    if up:
        xin = P.upsample_nearest2x(xin)
    if name == "3x3_big_tiles":
        # full size of the first level of the 768px model: compare sampled outputs computed one by one
        rng = np.random.default_rng(5)
        xp = np.pad(xin.astype(np.float64), ((0, 0), (0, 0), (1, 1), (1, 1)))
        errs, refs = [], []
        for _ in range(400):
            b, o, i, j = int(rng.integers(n)), int(rng.integers(n_out)), int(rng.integers(ho)), int(rng.integers(wo))
            ref = bias[o] + float(np.sum(w[o].astype(np.float64) * xp[b, :, i:i + 3, j:j + 3]))
            errs.append(got[b, i, j, o] - ref); refs.append(ref)
        assert_kernel_close(np.asarray(refs) + np.asarray(errs), np.asarray(refs), dtype)
        assert np.isfinite(got).all()
        return
    ref = P.conv2d(xin, w, bias, stride=stride)
    assert got.shape == (n, ho, wo, n_out)
    assert_kernel_close(nhwc_to_nchw(got), ref, dtype)


@pytest.mark.parametrize("dtype", DT)
def test_conv_epilogues(dtype):
    n, c, h, wd, n_out = 2, 64, 9, 7, 192
    x = quantize(SI.make_array((n, c, h, wd), 21), dtype)
    w = quantize(SI.make_array((n_out, c, 3, 3), 22, 0.05), dtype)
    bias = SI.make_array((n_out,), 23, 0.1)
    rowvec = SI.make_array((n, n_out), 24)
    res = quantize(SI.make_array((n, h, wd, n_out), 25), dtype)
    got, _ = run_conv(dtype, x, None, w, bias, rowvec=rowvec, residual=res)
    ref = P.conv2d(x, w, bias) + rowvec[:, :, None, None] + nhwc_to_nchw(res)
    assert_kernel_close(nhwc_to_nchw(got), ref, dtype)
    # transposed outputs (storage dtype and fp32)
    for mode in (B.OUT_TRANSPOSED, B.OUT_TRANSPOSED_F32):
        got, (ho, wo) = run_conv(dtype, x, None, w, bias, mode=mode)
        ref = P.conv2d(x, w, bias).reshape(n, n_out, ho * wo)
        assert_kernel_close(got[:, :, :ho * wo], ref, dtype)


@pytest.fixture(params=[1, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12], ids=["reg128", "reg64", "dma2_128", "dma3_128", "dma3_256", "dma3_64", "halo_128", "halo_256", "dma3_256_w4", "dma3_128_w4", "dma3_256_w16"])
def force_big_tiles(request):
    """Forces one GEMM kernel family on every shape (the LDS-DMA ones apply to bf16 only; fp32 keeps the automatic choice)."""
    B.check(lib.ad_tune_conv_tile(request.param))
    yield
    B.check(lib.ad_tune_conv_tile(-1))


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("case", CONV_CASES[:5], ids=[c[0] for c in CONV_CASES[:5]])
def test_conv_big_tile_kernels(dtype, case, force_big_tiles):
    test_conv_matches_direct_summation(dtype, case)
    test_conv_epilogues(dtype)
    test_linear_and_geglu(dtype)
    test_conv_split_k(dtype)


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("big", [0, 1, 4, 5, 6, 7, 10, 11, 12])
@pytest.mark.parametrize("vt", [False, True])
def test_fused_qkv_projection(dtype, big, vt):
    """One GEMM for q, k, v: thirds of the output columns go to three tensors, the last optionally transposed."""
    bsz, l, c = 2, 72, 64
    if big:
        B.check(lib.ad_tune_conv_tile(big))
    try:
        x = quantize(SI.make_array((bsz * l, c), 35), dtype)
        w = quantize(SI.make_array((3 * c, c), 36, 0.2), dtype)
        dx = dev(x, dtype)
        wp = dev_bytes(B.pack_conv_weight(dtype, w))
        ld_t = 128 if vt else 0
        q = torch.full((bsz * l, c), float("nan"), device=DEV, dtype=tdtype(dtype))
        k = torch.full((bsz * l, c), float("nan"), device=DEV, dtype=tdtype(dtype))
        v = torch.full((bsz, c, ld_t) if vt else (bsz * l, c), float("nan"), device=DEV, dtype=tdtype(dtype))
        B.check(lib.ad_conv_forward(dtype, p(dx), None, c, 0, bsz, l, 1, 0, 1, 1, p(wp), 3 * c, None, None, None, p(q), p(k), p(v),
                                    B.OUT_QKV, ld_t, None, 0, stream_ptr()))
        sync()
    finally:
        B.check(lib.ad_tune_conv_tile(-1))
    ref = P.linear(x, w)
    assert_kernel_close(host(q), ref[:, :c], dtype)
    assert_kernel_close(host(k), ref[:, c:2 * c], dtype)
    if vt:
        got = host(v)[:, :, :l]
        assert_kernel_close(got, ref[:, 2 * c:].reshape(bsz, l, c).transpose(0, 2, 1), dtype)
    else:
        assert_kernel_close(host(v), ref[:, 2 * c:], dtype)


@pytest.mark.parametrize("dtype", DT)
def test_conv_split_k(dtype):
    """Deep-level shapes (few output positions, long K) take the split-K path when scratch is supplied."""
    n, c, h, wd, n_out = 2, 640, 6, 6, 192
    x = quantize(SI.make_array((n, c, h, wd), 26), dtype)
    w = quantize(SI.make_array((n_out, c, 3, 3), 27, 0.02), dtype)
    bias = SI.make_array((n_out,), 28, 0.1)
    rowvec = SI.make_array((n, n_out), 29)
    res = quantize(SI.make_array((n, h, wd, n_out), 30), dtype)
    ref = P.conv2d(x, w, bias) + rowvec[:, :, None, None] + nhwc_to_nchw(res)
    got, _ = run_conv(dtype, x, None, w, bias, rowvec=rowvec, residual=res, splitk=True)
    assert run_conv.last_ws_bytes > 0, "shape was expected to split"
    assert_kernel_close(nhwc_to_nchw(got), ref, dtype)
    plain, _ = run_conv(dtype, x, None, w, bias, rowvec=rowvec, residual=res, splitk=False)
    assert_kernel_close(nhwc_to_nchw(plain), ref, dtype)
    got, (ho, wo) = run_conv(dtype, x, None, w, bias, mode=B.OUT_TRANSPOSED_F32, splitk=True)
    assert_kernel_close(got[:, :, :ho * wo], P.conv2d(x, w, bias).reshape(n, n_out, ho * wo), dtype)


EDGE_TILES = [-1, 1, 3, 4, 5, 6, 7, 14, 15]


@pytest.mark.parametrize("tile", EDGE_TILES)
@pytest.mark.parametrize("n_out,shift", [(192, 0), (192, 4), (200, 0), (36, 0), (68, 4), (130, 0), (328, 0)])
def test_gemm_epilogue_widths_and_alignment(tile, n_out, shift):
    """Row-major output with bias, per-sample vector and residual: rows of whole 16-byte groups, of whole 8-byte groups and of single
    elements, tensors that start off a 16-byte boundary, tiles that span three samples and tiles inside one."""
    for n, h, wd in ((2, 16, 18), (5, 7, 9)):
        c = 128
        x = quantize(SI.make_array((n, c, h, wd), 341), B.AD_BF16)
        w = quantize(SI.make_array((n_out, c, 3, 3), 342, 0.05), B.AD_BF16)
        bias, rowvec = SI.make_array((n_out,), 343, 0.1), SI.make_array((n, n_out), 344)
        res = quantize(SI.make_array((n, h, wd, n_out), 345), B.AD_BF16)
        dx, wp = dev(nchw_to_nhwc(x), B.AD_BF16), dev_bytes(B.pack_conv_weight(B.AD_BF16, w))
        size = n * h * wd * n_out
        out, dres = (torch.full((size + 16,), float("nan"), device=DEV, dtype=torch.bfloat16) for _ in range(2))
        dres[shift:shift + size] = dev(res, B.AD_BF16).reshape(-1)
        db, dv = dev(bias, B.AD_F32), dev(rowvec, B.AD_F32)
        B.check(lib.ad_tune_conv_tile(tile))
        try:
            B.check(lib.ad_conv_forward(B.AD_BF16, p(dx), None, c, 0, n, h, wd, 0, 3, 1, p(wp), n_out, p(db), p(dv), p(dres[shift:]), p(out[shift:]),
                                        None, None, B.OUT_ROWMAJOR, 0, None, 0, stream_ptr()))
            sync()
        finally:
            B.check(lib.ad_tune_conv_tile(-1))
        got = host(out)
        assert np.isnan(got[:shift]).all() and np.isnan(got[shift + size:]).all()
        ref = P.conv2d(x, w, bias) + rowvec[:, :, None, None] + nhwc_to_nchw(res)
        assert_kernel_close(nhwc_to_nchw(got[shift:shift + size].reshape(n, h, wd, n_out)), ref, B.AD_BF16)


@pytest.mark.parametrize("tile", EDGE_TILES)
@pytest.mark.parametrize("bsz,l,c,ld_t,shift", [(2, 72, 64, 72, 0), (2, 72, 64, 76, 0), (3, 44, 64, 48, 0), (3, 45, 64, 45, 0), (1, 300, 320, 304, 0), (2, 72, 64, 72, 4), (2, 136, 96, 136, 0)])
def test_qkv_transposed_third(tile, bsz, l, c, ld_t, shift):
    """The transposed third of the fused projection: whole 16-byte groups of rows, sample lengths and pitches that are not, tiles
    across samples, a destination off a 16-byte boundary; thirds of 96 columns share a 64-column slab."""
    cin = 64
    x = quantize(SI.make_array((bsz * l, cin), 351), B.AD_BF16)
    w = quantize(SI.make_array((3 * c, cin), 352, 0.2), B.AD_BF16)
    dx, wp = dev(x, B.AD_BF16), dev_bytes(B.pack_conv_weight(B.AD_BF16, w))
    q, k = (torch.full((bsz * l, c), float("nan"), device=DEV, dtype=torch.bfloat16) for _ in range(2))
    v = torch.full((bsz * c * ld_t + 16,), float("nan"), device=DEV, dtype=torch.bfloat16)
    B.check(lib.ad_tune_conv_tile(tile))
    try:
        B.check(lib.ad_conv_forward(B.AD_BF16, p(dx), None, cin, 0, bsz, l, 1, 0, 1, 1, p(wp), 3 * c, None, None, None, p(q), p(k), p(v[shift:]),
                                    B.OUT_QKV, ld_t, None, 0, stream_ptr()))
        sync()
    finally:
        B.check(lib.ad_tune_conv_tile(-1))
    ref = P.linear(x, w)
    assert_kernel_close(host(q), ref[:, :c], B.AD_BF16)
    assert_kernel_close(host(k), ref[:, c:2 * c], B.AD_BF16)
    got = host(v)[shift:shift + bsz * c * ld_t].reshape(bsz, c, ld_t)
    assert_kernel_close(got[:, :, :l], ref[:, 2 * c:].reshape(bsz, l, c).transpose(0, 2, 1), B.AD_BF16)
    assert np.isnan(got[:, :, l:]).all()


@pytest.mark.parametrize("tile", [14, 15])
@pytest.mark.parametrize("case", CONV_CASES[:5] + [None], ids=[c[0] for c in CONV_CASES[:5]] + ["epilogues"])
def test_conv_wide_tiles(tile, case):
    B.check(lib.ad_tune_conv_tile(tile))
    try:
        if case:
            test_conv_matches_direct_summation(B.AD_BF16, case)
        else:
            test_conv_epilogues(B.AD_BF16)
            test_conv_split_k(B.AD_BF16)
    finally:
        B.check(lib.ad_tune_conv_tile(-1))


@pytest.mark.parametrize("tile", [-1, 4, 5, 6, 15])
@pytest.mark.parametrize("rows,cin,cff", [(300, 64, 160), (77, 128, 32), (520, 64, 224), (256, 192, 64), (130, 64, 96)])
def test_geglu_tile_edges(tile, rows, cin, cff):
    """Projection widths that end in every value / gate pair of a 320-column tile (one of them is shared by two wavefronts); a gate far
    out on either side."""
    x = quantize(SI.make_array((1, cin, rows, 1), 361), B.AD_BF16)
    w = quantize(SI.make_array((2 * cff, cin), 362, 0.2), B.AD_BF16)
    b = SI.make_array((2 * cff,), 363, 0.1)
    b[cff:cff + 4] = (40.0, -40.0, 300.0, -300.0)
    B.check(lib.ad_tune_conv_tile(tile))
    try:
        got, _ = run_conv(B.AD_BF16, x, None, w[:, :, None, None], b, mode=B.OUT_GEGLU, geglu=True)
    finally:
        B.check(lib.ad_tune_conv_tile(-1))
    y = P.linear(x[0, :, :, 0].T, w, b)
    ref = y[:, :cff] * P.gelu(y[:, cff:])
    assert_kernel_close(got.reshape(rows, cff), ref, B.AD_BF16)


@pytest.mark.parametrize("tile", [4, 14, 15])
@pytest.mark.parametrize("c0,c1,k,stride,up", [(192, 64, 3, 1, 1), (64, 192, 3, 2, 0), (128, 128, 1, 2, 0), (64, 64, 3, 1, 0)])
def test_two_stage_tiles_follow_sources_and_taps(tile, c0, c1, k, stride, up):
    """The change of source in the middle of a tap, strides and a nearest-2x input of odd size, split over K or not."""
    n, hs, ws, n_out = 2, 9, 7, 96
    x0, x1 = (quantize(SI.make_array((n, c, hs, ws), 371 + i), B.AD_BF16) for i, c in enumerate((c0, c1)))
    w = quantize(SI.make_array((n_out, c0 + c1, k, k), 373, 0.05), B.AD_BF16)
    bias = SI.make_array((n_out,), 374, 0.1)
    xin = np.concatenate([x0, x1], 1)
    ref = P.conv2d(P.upsample_nearest2x(xin) if up else xin, w, bias, stride=stride)
    B.check(lib.ad_tune_conv_tile(tile))
    try:
        for splitk in (False, True):
            got, _ = run_conv(B.AD_BF16, x0, x1, w, bias, stride, up, splitk=splitk)
            assert_kernel_close(nhwc_to_nchw(got), ref, B.AD_BF16)
    finally:
        B.check(lib.ad_tune_conv_tile(-1))


@pytest.mark.parametrize("rows,cin,n_out,tile", [(2048, 128, 1280, 5), (1800, 128, 1100, 5), (4500, 64, 640, 6), (1100, 448, 448, 7), (1100, 448, 448, -1), (2900, 64, 800, 14),
                                                 (3000, 64, 1600, 15), (900, 1024, 640, 4), (4096, 64, 1280, 5), (2100, 64, 3840, 6)])
def test_workgroup_order_in_bands(rows, cin, n_out, tile):
    """Every output tile once, whatever the order: bands of several row tiles with a shorter last one, runs of an XCD that end inside a band, K-splits,
    several rounds of which the bands are not to begin at the same column everywhere.
    The order changes no sum, so all three are equal bit for bit."""
    x, w = quantize(SI.make_array((rows, cin), 71), B.AD_BF16), quantize(SI.make_array((n_out, cin), 72, 0.1), B.AD_BF16)
    got = []
    B.check(lib.ad_tune_conv_tile(tile))
    try:
        for order in (-1, 0, 1):
            B.check(lib.ad_tune_conv_order(order))
            got.append(run_conv(B.AD_BF16, x.T.reshape(1, cin, rows, 1), None, w.reshape(n_out, cin, 1, 1), None, splitk=True)[0].reshape(rows, n_out))
    finally:
        B.check(lib.ad_tune_conv_tile(-1))
        B.check(lib.ad_tune_conv_order(-1))
    assert_kernel_close(got[0], P.linear(x, w), B.AD_BF16)
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])


@pytest.mark.parametrize("c0,c1,k,stride,up,n_out", [(448, 0, 1, 1, 0, 640), (64, 0, 3, 1, 0, 640), (128, 64, 3, 1, 0, 600), (640, 640, 1, 1, 0, 642),
                                                     (192, 0, 3, 2, 0, 1280), (64, 128, 3, 1, 1, 320), (2496, 0, 1, 1, 0, 640)])
def test_k_shared_by_two_groups(c0, c1, k, stride, up, n_out):
    """64x64 tiles whose k-tiles are shared out over two groups of wavefronts: odd and even numbers of k-tiles, changes of tap and source at and beside
    the middle, ragged rows and columns, everything the epilogue adds."""
    n, hs, ws = (2, 25, 20) if not up else (2, 12, 11)
    x0, x1 = (quantize(SI.make_array((n, c, hs, ws), 391 + i), B.AD_BF16) if c else None for i, c in enumerate((c0, c1)))
    w = quantize(SI.make_array((n_out, c0 + c1, k, k), 393, 0.05), B.AD_BF16)
    bias, rowvec = SI.make_array((n_out,), 394, 0.1), SI.make_array((n, n_out), 395)
    xin = x0 if x1 is None else np.concatenate([x0, x1], 1)
    ref = P.conv2d(P.upsample_nearest2x(xin) if up else xin, w, bias, stride=stride) + rowvec[:, :, None, None]
    res = quantize(SI.make_array((n, ref.shape[2], ref.shape[3], n_out), 396), B.AD_BF16)
    for tile, splitk in ((16, False), (-1, False), (-1, True)):
        B.check(lib.ad_tune_conv_tile(tile))
        try:
            got, _ = run_conv(B.AD_BF16, x0, x1, w, bias, stride, up, rowvec=rowvec, residual=res, splitk=splitk)
        finally:
            B.check(lib.ad_tune_conv_tile(-1))
        assert_kernel_close(nhwc_to_nchw(got), ref + nhwc_to_nchw(res), B.AD_BF16)


@pytest.mark.parametrize("hs,ws,c0,c1,k,n_out,last", [(8, 4, 2368, 0, 1, 64, 2), (8, 4, 2112, 0, 1, 52, 3), (8, 4, 256, 256, 3, 64, 2), (7, 4, 320, 128, 3, 64, 3),
                                                      (8, 4, 704, 0, 3, 36, 3)])
def test_k_shared_by_workgroups_and_two_groups_each(hs, ws, c0, c1, k, n_out, last):
    """The same with K shared out over workgroups first: the last of them has two or three k-tiles, one for each group of wavefronts or one more."""
    x0, x1 = (quantize(SI.make_array((2, c, hs, ws), 411 + i), B.AD_BF16) if c else None for i, c in enumerate((c0, c1)))
    w, bias = quantize(SI.make_array((n_out, c0 + c1, k, k), 413, 0.05), B.AD_BF16), SI.make_array((n_out,), 414, 0.1)
    B.check(lib.ad_tune_conv_tile(16))
    try:
        got, _ = run_conv(B.AD_BF16, x0, x1, w, bias, splitk=True)
    finally:
        B.check(lib.ad_tune_conv_tile(-1))
    ktiles, splits = k * k * (c0 + c1) // 64, run_conv.last_ws_bytes // (2 * hs * ws * n_out * 4)
    assert splits > 1 and ktiles - (splits - 1) * -(-ktiles // splits) == last, (ktiles, splits)
    assert_kernel_close(nhwc_to_nchw(got), P.conv2d(x0 if x1 is None else np.concatenate([x0, x1], 1), w, bias), B.AD_BF16)


@pytest.mark.parametrize("l,c,cin,ld_t", [(500, 320, 640, 512), (333, 192, 704, 0), (257, 320, 1344, 260)])
def test_k_shared_by_two_groups_fused_projection(l, c, cin, ld_t):
    x, w = quantize(SI.make_array((2 * l, cin), 397), B.AD_BF16), quantize(SI.make_array((3 * c, cin), 398, 0.05), B.AD_BF16)
    dx, wp = dev(x, B.AD_BF16), dev_bytes(B.pack_conv_weight(B.AD_BF16, w))
    q, k = (torch.full((2 * l, c), float("nan"), device=DEV, dtype=torch.bfloat16) for _ in range(2))
    v = torch.full((2 * c * ld_t if ld_t else 2 * l * c,), float("nan"), device=DEV, dtype=torch.bfloat16)
    B.check(lib.ad_tune_conv_tile(16))
    try:
        B.check(lib.ad_conv_forward(B.AD_BF16, p(dx), None, cin, 0, 2, l, 1, 0, 1, 1, p(wp), 3 * c, None, None, None, p(q), p(k), p(v), B.OUT_QKV, ld_t, None, 0,
                                    stream_ptr()))
        sync()
    finally:
        B.check(lib.ad_tune_conv_tile(-1))
    ref = P.linear(x, w)
    assert_kernel_close(host(q), ref[:, :c], B.AD_BF16)
    assert_kernel_close(host(k), ref[:, c:2 * c], B.AD_BF16)
    got = host(v).reshape(2, c, ld_t)[:, :, :l] if ld_t else host(v).reshape(2, l, c).transpose(0, 2, 1)
    assert_kernel_close(got, ref[:, 2 * c:].reshape(2, l, c).transpose(0, 2, 1), B.AD_BF16)


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("tile", [-1, 5, 14])
@pytest.mark.parametrize("bsz,l,c,ld_t,shift", [(2, 36, 64, 0, 0), (2, 36, 64, 0, 1), (2, 36, 64, 36, 0), (3, 21, 96, 21, 2), (1, 70, 32, 96, 4)])
def test_split_k_second_pass_of_the_fused_projection(dtype, tile, bsz, l, c, ld_t, shift):
    """The thirds of q/k/v out of partial sums: row-major and transposed, whole vectors and single elements, destinations off a vector."""
    cin = 5120
    x = quantize(SI.make_array((bsz * l, cin), 381), dtype)
    w = quantize(SI.make_array((3 * c, cin), 382, 0.02), dtype)
    dx, wp = dev(x, dtype), dev_bytes(B.pack_conv_weight(dtype, w))
    q, k = (torch.full((bsz * l * c + 8,), float("nan"), device=DEV, dtype=tdtype(dtype)) for _ in range(2))
    size = bsz * c * ld_t if ld_t else bsz * l * c
    v = torch.full((size + 8,), float("nan"), device=DEV, dtype=tdtype(dtype))
    B.check(lib.ad_tune_conv_tile(tile))
    try:
        ws_bytes = lib.ad_conv_workspace_bytes(dtype, bsz, l, 1, 3 * c, cin, 1, B.OUT_QKV)
        assert ws_bytes > 0, "shape was expected to split"
        wsb = torch.zeros(ws_bytes, dtype=torch.uint8, device=DEV)
        B.check(lib.ad_conv_forward(dtype, p(dx), None, cin, 0, bsz, l, 1, 0, 1, 1, p(wp), 3 * c, None, None, None, p(q[shift:]), p(k[shift:]),
                                    p(v[shift:]), B.OUT_QKV, ld_t, p(wsb), ws_bytes, stream_ptr()))
        sync()
    finally:
        B.check(lib.ad_tune_conv_tile(-1))
    ref = P.linear(x, w)
    for t, r in ((q, ref[:, :c]), (k, ref[:, c:2 * c])):
        got = host(t)
        assert np.isnan(got[:shift]).all() and np.isnan(got[shift + r.size:]).all()
        assert_kernel_close(got[shift:shift + r.size].reshape(r.shape), r, dtype)
    got = host(v)
    assert np.isnan(got[:shift]).all() and np.isnan(got[shift + size:]).all()
    got = got[shift:shift + size]
    if ld_t:
        got = got.reshape(bsz, c, ld_t)
        assert np.isnan(got[:, :, l:]).all()
        assert_kernel_close(got[:, :, :l], ref[:, 2 * c:].reshape(bsz, l, c).transpose(0, 2, 1), dtype)
    else:
        assert_kernel_close(got.reshape(bsz * l, c), ref[:, 2 * c:], dtype)


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("mode", [B.OUT_ROWMAJOR, B.OUT_TRANSPOSED, B.OUT_TRANSPOSED_F32], ids=["rows", "turned", "turned_f32"])
@pytest.mark.parametrize("n_out,shift", [(192, 0), (36, 0), (200, 1), (68, 2), (192, 4)])
def test_split_k_second_pass_alignment(dtype, mode, n_out, shift):
    """Bias, per-sample vector and (row-major) residual added to partial sums, tensors on and off a boundary of four elements."""
    n, c, h, wd = 2, 640, 5, 7
    x = quantize(SI.make_array((n, c, h, wd), 391), dtype)
    w = quantize(SI.make_array((n_out, c, 3, 3), 392, 0.02), dtype)
    bias, rowvec = SI.make_array((n_out,), 393, 0.1), SI.make_array((n, n_out), 394)
    ref = P.conv2d(x, w, bias) + rowvec[:, :, None, None]
    ld_t, size = (0, n * h * wd * n_out) if mode == B.OUT_ROWMAJOR else (h * wd + 2, n * n_out * (h * wd + 2))
    dres = None
    if mode == B.OUT_ROWMAJOR:
        res = quantize(SI.make_array((n, h, wd, n_out), 395), dtype)
        ref = ref + nhwc_to_nchw(res)
        dres = torch.full((size + 8,), float("nan"), device=DEV, dtype=tdtype(dtype))
        dres[shift:shift + size] = dev(res, dtype).reshape(-1)
        dres = dres[shift:]
    out = torch.full((size + 8,), float("nan"), device=DEV, dtype=torch.float32 if mode == B.OUT_TRANSPOSED_F32 else tdtype(dtype))
    dx, wp, db, dv = dev(nchw_to_nhwc(x), dtype), dev_bytes(B.pack_conv_weight(dtype, w)), dev_f32(bias), dev_f32(rowvec)
    ws_bytes = lib.ad_conv_workspace_bytes(dtype, n, h, wd, n_out, c, 3, mode)
    assert ws_bytes > 0, "shape was expected to split"
    wsb = torch.zeros(ws_bytes, dtype=torch.uint8, device=DEV)
    B.check(lib.ad_conv_forward(dtype, p(dx), None, c, 0, n, h, wd, 0, 3, 1, p(wp), n_out, p(db), p(dv), p(dres), p(out[shift:]), None, None,
                                mode, ld_t, p(wsb), ws_bytes, stream_ptr()))
    sync()
    got = host(out)
    assert np.isnan(got[:shift]).all() and np.isnan(got[shift + size:]).all()
    got = got[shift:shift + size]
    if mode == B.OUT_ROWMAJOR:
        assert_kernel_close(nhwc_to_nchw(got.reshape(n, h, wd, n_out)), ref, dtype)
    else:
        got = got.reshape(n, n_out, ld_t)
        assert np.isnan(got[:, :, h * wd:]).all()
        assert_kernel_close(got[:, :, :h * wd], ref.reshape(n, n_out, h * wd), dtype)


SMALL_CASES = [
    # edges of the small-tile kernel: one row, fewer k-tiles than wavefronts, 16x16 / 16x32 / 32x32 tiles with remainders, K that does
    # not divide over the wavefronts, two sources, stride 2, nearest-2x input with odd sizes, few columns
    ("one_row", 1, 64, 0, 1, 1, 64, 1, 1, 0), ("one_tile_k", 1, 64, 0, 5, 3, 20, 1, 1, 0), ("16x16_ragged", 2, 128, 0, 7, 9, 132, 3, 1, 0),
    ("16x32_ragged", 2, 64, 0, 23, 24, 72, 3, 1, 0), ("32x32_ragged", 1, 320, 0, 13, 21, 520, 1, 1, 0), ("concat", 1, 64, 128, 11, 6, 96, 3, 1, 0),
    ("stride2", 2, 64, 0, 14, 10, 64, 3, 2, 0), ("stride2_1x1", 1, 128, 0, 9, 9, 48, 1, 2, 0), ("up", 2, 64, 64, 5, 7, 64, 3, 1, 1),
    ("few_columns", 2, 64, 0, 12, 12, 4, 3, 1, 0), ("odd_columns", 1, 64, 0, 6, 6, 7, 3, 1, 0),
    # maps smaller than the distance between the first and the last tap: one pixel, one row, one column, of one sample and of two
    ("one_pixel", 1, 256, 0, 1, 1, 256, 3, 1, 0), ("one_pixel_x2", 2, 256, 0, 1, 1, 256, 3, 1, 0), ("one_pixel_concat", 2, 64, 128, 1, 1, 64, 3, 1, 0),
    ("one_row_3x3", 1, 128, 0, 1, 6, 96, 3, 1, 0), ("one_row_concat", 1, 64, 64, 1, 5, 64, 3, 1, 0), ("one_column", 1, 128, 0, 2, 1, 64, 3, 1, 0),
    ("one_row_stride2", 1, 64, 0, 1, 9, 64, 3, 2, 0), ("one_pixel_up", 1, 128, 0, 1, 1, 64, 3, 1, 1),
]


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("case", SMALL_CASES, ids=[c[0] for c in SMALL_CASES])
def test_conv_small_tiles(dtype, case):
    """Row-major (bias, per-sample vector, residual) and both transposed outputs of one shape."""
    name, n, c0, c1, hs, ws, n_out, k, stride, up = case
    x0 = quantize(SI.make_array((n, c0, hs, ws), 311), dtype)
    x1 = quantize(SI.make_array((n, c1, hs, ws), 312), dtype) if c1 else None
    w = quantize(SI.make_array((n_out, c0 + c1, k, k), 313, 0.05), dtype)
    bias, rowvec = SI.make_array((n_out,), 314, 0.1), SI.make_array((n, n_out), 315)
    xin = x0 if x1 is None else np.concatenate([x0, x1], 1)
    ref = P.conv2d(P.upsample_nearest2x(xin) if up else xin, w, bias, stride=stride)
    ho, wo = ref.shape[2:]
    res = quantize(SI.make_array((n, ho, wo, n_out), 316), dtype)
    got, _ = run_conv(dtype, x0, x1, w, bias, stride, up, rowvec=rowvec, residual=res)
    assert_kernel_close(nhwc_to_nchw(got), ref + rowvec[:, :, None, None] + nhwc_to_nchw(res), dtype)
    for mode in (B.OUT_TRANSPOSED, B.OUT_TRANSPOSED_F32):
        got, _ = run_conv(dtype, x0, x1, w, bias, stride, up, mode=mode)
        assert_kernel_close(got[:, :, :ho * wo], ref.reshape(n, n_out, ho * wo), dtype)


@pytest.mark.parametrize("dtype", DT)
def test_linear_and_geglu(dtype):
    rows, cin, cff = 200, 64, 256                      # GEGLU: 64 -> 2*256, value * gelu(gate)
    x = quantize(SI.make_array((1, cin, rows, 1), 31), dtype)
    w1 = quantize(SI.make_array((2 * cff, cin), 32, 0.2), dtype)
    b1 = SI.make_array((2 * cff,), 33, 0.1)
    got, _ = run_conv(dtype, x, None, w1[:, :, None, None], b1, mode=B.OUT_GEGLU, geglu=True)
    tok = x[0, :, :, 0].T
    hcat = P.linear(tok, w1, b1)
    ref = hcat[:, :cff] * P.gelu(hcat[:, cff:])
    assert_kernel_close(got.reshape(rows, cff), ref, dtype)
    w2 = quantize(SI.make_array((96, cin), 34, 0.2), dtype)
    got, _ = run_conv(dtype, x, None, w2[:, :, None, None], None)
    assert_kernel_close(got.reshape(rows, 96), P.linear(tok, w2), dtype)


# ---------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("shape", [(2, 64, 0, 16, 16, 8, 1), (2, 320, 0, 24, 24, 32, 1), (1, 64, 32, 9, 7, 8, 0),
                                   (2, 640, 320, 12, 12, 32, 1), (2, 2560, 0, 6, 6, 32, 1)])
def test_groupnorm_silu(dtype, shape):
    n, c0, c1, h, w, groups, silu = shape
    x0 = quantize(SI.make_array((n, c0, h, w), 41) * 2 + 0.5, dtype)
    x1 = quantize(SI.make_array((n, c1, h, w), 42) - 1.0, dtype) if c1 else None
    gam, bet = 1 + SI.make_array((c0 + c1,), 43, 0.3), SI.make_array((c0 + c1,), 44, 0.3)
    d0 = dev(nchw_to_nhwc(x0), dtype)
    d1 = dev(nchw_to_nhwc(x1), dtype) if c1 else None
    out = torch.full((n, h, w, c0 + c1), float("nan"), device=DEV, dtype=tdtype(dtype))
    scratch = torch.zeros(lib.ad_groupnorm_scratch_bytes(n, h * w, c0 + c1), dtype=torch.uint8, device=DEV)
    dg, dbt = dev_f32(gam), dev_f32(bet)
    B.check(lib.ad_groupnorm_forward(dtype, p(d0), p(d1), c0, c1, n, h * w, groups, p(dg), p(dbt), 1e-5, silu, p(out), p(scratch), stream_ptr()))
    sync()
    xin = x0 if x1 is None else np.concatenate([x0, x1], 1)
    ref = P.group_norm(xin, groups, gam, bet, 1e-5)
    if silu:
        ref = P.silu(ref)
    assert_kernel_close(nhwc_to_nchw(host(out)), ref, dtype, rel=1e-5 if dtype == B.AD_F32 else 5e-3)


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("shape", [
    # one launch: 8 / 4 / 2 channels per access (4 / 2 / 1 in fp32), 256 / 512 / 1024 threads, few and many registers, one pixel,
    # a group that straddles the two sources
    (2, 256, 0, 1, 1, 32, 1), (1, 64, 0, 45, 23, 32, 1), (2, 128, 64, 24, 24, 32, 0), (1, 640, 0, 24, 21, 32, 1), (1, 1280, 640, 15, 17, 32, 1),
    (1, 1280, 0, 37, 23, 32, 1), (1, 320, 0, 40, 39, 32, 1), (2, 96, 64, 19, 19, 16, 1), (2, 320, 0, 43, 41, 32, 1), (4, 2560, 0, 27, 23, 32, 1),
    (9, 128, 0, 40, 39, 32, 1), (1, 1280, 0, 7, 5, 320, 1),
    # two launches: each limit of the choice exceeded, an odd number of channels per group (bf16), several sources and samples, more
    # than 256 channel vectors, few chunks, samples that do not divide the workgroups
    (2, 320, 0, 61, 59, 32, 1), (1, 2560, 0, 27, 29, 32, 1), (1, 640, 320, 48, 39, 32, 1), (2, 64, 96, 11, 5, 32, 0), (3, 64, 32, 9, 7, 32, 1),
    (1, 2560, 0, 83, 61, 128, 1), (1, 64, 0, 83, 61, 32, 1), (5, 320, 0, 61, 59, 32, 1), (9, 128, 64, 57, 55, 32, 1)])
def test_groupnorm_every_path(dtype, shape):
    test_groupnorm_silu(dtype, shape)


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("batch,c,hw,groups", [(1, 128, 1024, 32), (1, 128, 1023, 32), (1, 128, 2051, 32), (2, 320, 2049, 32), (2, 1280, 205, 32), (1, 64, 512, 8),
                                               (2, 64, 259, 1), (1, 1280, 3, 1), (4, 256, 1111, 32)])
def test_groupnorm_shared_by_workgroups_and_in_place(dtype, batch, c, hw, groups):
    """Groups of one launch whose result several workgroups write: around the lines between one, two and four of them, ragged last rounds, fewer rounds
    than workgroups; and the same call with its input as output, which leaves a group to one workgroup: the same bits."""
    x = quantize(SI.make_array((batch, hw, c), 48) * 2 + 0.5, dtype)
    gam, bet = 1 + SI.make_array((c,), 49, 0.3), SI.make_array((c,), 50, 0.3)
    ref = P.silu(P.group_norm(x.transpose(0, 2, 1)[..., None], groups, gam, bet, 1e-5))[..., 0].transpose(0, 2, 1)
    d, dg, dbt = dev(x, dtype), dev_f32(gam), dev_f32(bet)
    scratch = torch.zeros(lib.ad_groupnorm_scratch_bytes(batch, hw, c), dtype=torch.uint8, device=DEV)
    got = []
    for out in (torch.full_like(d, float("nan")), d):
        B.check(lib.ad_groupnorm_forward(dtype, p(d), None, c, 0, batch, hw, groups, p(dg), p(dbt), 1e-5, 1, p(out), p(scratch), stream_ptr()))
        sync()
        got.append(host(out))
        assert_kernel_close(got[-1], ref, dtype, rel=1e-5 if dtype == B.AD_F32 else 5e-3)
    assert np.array_equal(got[0], got[1])


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("shape", [(2, 256, 0, 6, 7, 32), (1, 640, 320, 24, 21, 32), (2, 1280, 0, 24, 24, 32), (2, 320, 0, 61, 59, 32), (1, 4608, 0, 9, 7, 32)],
                         ids=["one_launch_256", "one_launch_straddling", "one_launch_1024", "two_launches", "4608_channels"])
@pytest.mark.parametrize("outlier,offset", [(30.0, 0.0), (-100.0, 0.0), (0.0, 10.0), (0.0, -100.0)])
def test_groupnorm_outliers_and_offsets(dtype, shape, outlier, offset):
    """Statistics that must not cancel: the first element of every group of every sample far out, all elements far from zero."""
    n, c0, c1, h, w, groups = shape
    if h * w > 3000 and abs(offset) > 10:
        offset = math.copysign(10.0, offset)       # two launches: fp32 sums of squares about zero, 2^-24 (1 + offset^2) at most
    c = c0 + c1
    x = SI.make_array((n, c, h, w), 45) + offset
    if outlier:
        x[:, ::c // groups, 0, 0] = outlier
    x = quantize(x, dtype)
    gam, bet = 1 + SI.make_array((c,), 46, 0.3), SI.make_array((c,), 47, 0.3)
    d0, d1 = dev(nchw_to_nhwc(x[:, :c0]), dtype), dev(nchw_to_nhwc(x[:, c0:]), dtype) if c1 else None
    out = torch.full((n, h, w, c), float("nan"), device=DEV, dtype=tdtype(dtype))
    scratch = torch.zeros(lib.ad_groupnorm_scratch_bytes(n, h * w, c), dtype=torch.uint8, device=DEV)
    dg, dbt = dev_f32(gam), dev_f32(bet)
    B.check(lib.ad_groupnorm_forward(dtype, p(d0), p(d1), c0, c1, n, h * w, groups, p(dg), p(dbt), 1e-5, 0, p(out), p(scratch), stream_ptr()))
    sync()
    assert_kernel_close(nhwc_to_nchw(host(out)), P.group_norm(x, groups, gam, bet, 1e-5), dtype, rel=1e-5 if dtype == B.AD_F32 else 5e-3)


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("rows,c", [(7, 64), (300, 320), (33, 1280)])
def test_layernorm(dtype, rows, c):
    x = quantize(SI.make_array((rows, c), 51) * 3 + 1, dtype)
    gam, bet = 1 + SI.make_array((c,), 52, 0.3), SI.make_array((c,), 53, 0.3)
    dx, out = dev(x, dtype), torch.full((rows, c), float("nan"), device=DEV, dtype=tdtype(dtype))
    dg, dbt = dev_f32(gam), dev_f32(bet)
    B.check(lib.ad_layernorm_forward(dtype, p(dx), rows, c, p(dg), p(dbt), 1e-5, p(out), stream_ptr()))
    sync()
    assert_kernel_close(host(out), P.layer_norm(x, gam, bet, 1e-5), dtype, rel=1e-5 if dtype == B.AD_F32 else 5e-3)


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("rows,c", [(1, 8), (5, 16), (3, 24), (9000, 320), (8193, 640), (2050, 1280), (700, 1304), (66, 2560), (2, 4096), (20000, 88), (70000, 8), (300, 640), (64, 1024), (2880, 1000), (1152, 2048)])
def test_layernorm_lane_groups(dtype, rows, c):
    """Every number of lanes per row, rows that do not fill the last wavefront, widths that do not fill the lanes."""
    if c > 2048 and dtype == B.AD_F32:
        c //= 2
    test_layernorm(dtype, rows, c)


# ---------------------------------------------------------------------------------------------------
LOG2E_F32 = np.float32(1.4426950408889634)


def mfma2_contract(q, d, variant, dtype, transposed, lk):
    """The second-generation MFMA attention kernels feed the matrix cores q * (log2(e) / sqrt(d)) rounded to bf16 (one
    more rounding than the first kernel, which scales the fp32 scores).  That operand rounding is part of the kernel's
    contract like the bf16 storage of q itself, so the oracle is given the same operand: returns the q (fp64) whose
    plain softmax(q k^T / sqrt(d)) equals 2^(q' k^T) for the rounded q'.  Other kernels: q unchanged."""
    second = variant in (1, 2, 3) or (variant == -1 and lk > 256)
    if not (second and dtype == B.AD_BF16 and d == 64 and transposed):
        return q
    c32 = np.float32(1.0) / np.sqrt(np.float32(d)) * LOG2E_F32
    qp = SI.round_to_bf16(q.astype(np.float32) * c32)
    return qp.astype(np.float64) * (math.log(2.0) * math.sqrt(d))


def run_attention(dtype, q, k, v, heads, transposed):
    bsz, l, c = q.shape
    lk = k.shape[1]
    d = c // heads
    dq, dk = dev(q, dtype), dev(k, dtype)
    if transposed:
        ldv = (lk + 63) // 64 * 64
        vt = np.full((bsz, c, ldv), np.nan, np.float32)          # the pad must never be read as data
        vt[:, :, :lk] = np.transpose(v, (0, 2, 1))
        dv = dev(vt, dtype)
    else:
        ldv = c
        dv = dev(v, dtype)
    out = torch.full((bsz, l, c), float("nan"), device=DEV, dtype=tdtype(dtype))
    B.check(lib.ad_attention_forward(dtype, p(dq), p(dk), p(dv), int(transposed), bsz, l, lk, c, d, c, c, ldv, c, p(out), stream_ptr()))
    sync()
    return host(out)


ATT_CASES = [
    # dtype, batch, l, lk, heads, d, transposed
    (B.AD_F32, 1, 64, 64, 4, 16, False), (B.AD_F32, 2, 37, 8, 2, 16, False), (B.AD_F32, 1, 70, 130, 1, 64, False),
    (B.AD_BF16, 2, 37, 77, 2, 16, False), (B.AD_BF16, 1, 20, 77, 1, 128, True),
    (B.AD_BF16, 2, 200, 200, 3, 64, True), (B.AD_BF16, 2, 144, 77, 2, 64, True), (B.AD_BF16, 1, 576, 576, 5, 64, True),
    (B.AD_BF16, 1, 130, 1, 1, 64, True),
]


@pytest.fixture(params=[-1, 0, 1, 2, 3], ids=["auto", "gen1", "gen2_q32", "gen2_q64", "gen2_pipelined"])
def attn_variant(request):
    """Forces one of the MFMA attention kernels (applies to bf16, head width 64, transposed v; other calls are unaffected)."""
    B.check(lib.ad_tune_attention(request.param))
    yield request.param
    B.check(lib.ad_tune_attention(-1))


ATT_CASES += [
    # several 256-query blocks with a ragged tail, several key tiles with a ragged tail
    (B.AD_BF16, 2, 600, 333, 2, 64, True), (B.AD_BF16, 1, 257, 64, 1, 64, True), (B.AD_BF16, 1, 31, 65, 2, 64, True),
    (B.AD_BF16, 1, 1024, 1024, 1, 64, True), (B.AD_BF16, 2, 96, 128, 1, 64, True),
]


@pytest.mark.parametrize("case", ATT_CASES, ids=[f"{'bf16' if c[0] else 'f32'}_l{c[2]}_lk{c[3]}_h{c[4]}_d{c[5]}_{'vt' if c[6] else 'v'}" for c in ATT_CASES])
def test_attention(case, attn_variant):
    dtype, bsz, l, lk, heads, d, tr = case
    if attn_variant >= 0 and not (dtype == B.AD_BF16 and d == 64 and tr):
        pytest.skip("the knob only selects among the bf16 MFMA kernels")
    c = heads * d
    q, k, v = (quantize(SI.make_array(s, sd), dtype) for s, sd in (((bsz, l, c), 61), ((bsz, lk, c), 62), ((bsz, lk, c), 63)))
    got = run_attention(dtype, q, k, v, heads, tr)
    q = mfma2_contract(q, d, attn_variant, dtype, tr, lk)
    # the probabilities are rounded to bf16 and the result is an average of v rows: its rms is well below that of the
    # v entries the errors are proportional to
    assert_kernel_close(got, P.attention(q, k, v, heads), dtype, c=4.0)


GENERIC_CASES = [
    # the generic kernel: head widths in every register class, not a multiple of four (element loads), one key, one more and one
    # less than a 16-key block and than the 128 keys of a turn of the eight wavefronts, queries that do not fill a block, v transposed
    (B.AD_F32, 1, 1, 1, 1, 16, False), (B.AD_F32, 2, 17, 15, 1, 8, False), (B.AD_F32, 1, 33, 127, 2, 32, False), (B.AD_F32, 1, 15, 129, 1, 64, False),
    (B.AD_F32, 1, 40, 257, 1, 128, False), (B.AD_F32, 2, 19, 50, 3, 18, False), (B.AD_F32, 1, 21, 33, 5, 5, False), (B.AD_F32, 1, 48, 70, 1, 72, True),
    (B.AD_BF16, 1, 31, 65, 2, 40, False), (B.AD_BF16, 1, 18, 144, 3, 6, False), (B.AD_BF16, 1, 50, 30, 2, 64, False),
]


@pytest.mark.parametrize("case", GENERIC_CASES, ids=[f"{'bf16' if c[0] else 'f32'}_l{c[2]}_lk{c[3]}_h{c[4]}_d{c[5]}_{'vt' if c[6] else 'v'}" for c in GENERIC_CASES])
def test_attention_generic(case):
    test_attention(case, -1)


@pytest.mark.parametrize("dtype", DT)
@pytest.mark.parametrize("masked", [[(0, 16)], [(0, 48), (112, 144)], [(32, 300)], [(0, 299)]], ids=str)
def test_attention_generic_scores_of_minus_infinity(dtype, masked):
    """Keys whose score overflows to minus infinity have no weight, also where they are all that one wavefront sees for a while."""
    l, lk, d = 20, 300, 16
    q, k, v = (quantize(SI.make_array((1, n, d), 76 + i), dtype) for i, n in enumerate((l, lk, lk)))
    q[..., 0], k[..., 0] = quantize(1e20, dtype), 0.0
    keep = np.ones(lk, bool)
    for a, b in masked:
        keep[a:b] = False
    k[:, ~keep, 0] = quantize(-1e20, dtype)
    got = run_attention(dtype, q, k, v, 1, False)
    assert_kernel_close(got, P.attention(q, k[:, keep], v[:, keep], 1), dtype, c=4.0)


@pytest.mark.parametrize("dtype,tr", [(B.AD_F32, False), (B.AD_BF16, True)])
def test_attention_peaky_softmax(dtype, tr, attn_variant):
    """Scores far from uniform (scaled q, k) so that a mistake in the running max / rescaling shows."""
    bsz, l, lk, heads, d = 1, 96, 200, 2, 64
    c = heads * d
    q = quantize(SI.make_array((bsz, l, c), 71) * 3, dtype)
    k = quantize(SI.make_array((bsz, lk, c), 72) * 3, dtype)
    v = quantize(SI.make_array((bsz, lk, c), 73), dtype)
    # put the dominant key of some queries in the last tile so that the maximum moves late
    k[0, lk - 1] = q[0, 5] * 0.5
    got = run_attention(dtype, q, k, v, heads, tr)
    ref = P.attention(mfma2_contract(q, d, attn_variant, dtype, tr, lk), k, v, heads)
    assert_kernel_close(got, ref, dtype, c=4.0)
    pmax = P.softmax_rows(q[0, :, :d] @ k[0, :, :d].T / math.sqrt(d)).max(axis=1)
    assert np.median(pmax) > 0.5


@pytest.mark.parametrize("lk", [640, 700])
def test_attention_rising_and_falling_maximum(lk, attn_variant):
    """Scores that keep growing from key tile to key tile (the reference maximum has to move again and again, by
    more and by less than the slack the lazy maximum allows), then collapse far below it; one query row is all zeros."""
    dtype, l, d = B.AD_BF16, 300, 64
    rng = np.random.default_rng(77)
    base = rng.standard_normal((l, d)).astype(np.float32)
    q = quantize(base[None] * 2.0, dtype)
    q[0, 7] = 0.0
    k = rng.standard_normal((1, lk, d)).astype(np.float32) * 0.3
    ramp = np.concatenate([np.linspace(0.0, 3.0, lk // 2), np.linspace(3.0, -3.0, lk - lk // 2)]).astype(np.float32)
    k[0] += ramp[:, None] * np.sign(base[rng.integers(0, l, lk)])          # every key lines up with some query, more and more
    k = quantize(k, dtype)
    v = quantize(SI.make_array((1, lk, d), 75), dtype)
    got = run_attention(dtype, q, k, v, 1, True)
    ref = P.attention(mfma2_contract(q, d, attn_variant, dtype, True, lk), k, v, 1)
    assert_kernel_close(got, ref, dtype, c=4.0)
    sc = q[0] @ k[0].T / math.sqrt(d) * math.log2(math.e)
    tile_max = np.stack([sc[:, t:t + 32].max(axis=1) for t in range(0, lk, 32)], 1)
    run_max = np.maximum.accumulate(tile_max, axis=1)
    jumps = np.diff(run_max, axis=1)
    assert (jumps > 8).any() and ((jumps > 0) & (jumps < 8)).any()          # both kinds of moves occur


@pytest.mark.parametrize("bsz,l,lk,heads", [(1, 1, 257, 1), (2, 63, 320, 1), (1, 64, 321, 3), (1, 65, 383, 2), (2, 129, 384, 1), (1, 200, 1025, 1), (1, 70, 2111, 1)])
@pytest.mark.parametrize("ramp", [0.0, 6.0, -6.0])
def test_attention_keys_shared_out(bsz, l, lk, heads, ramp):
    """Launches of few queries share the keys out over two groups of wavefronts: query and key counts around the tiles, even and odd
    numbers of tiles, and scores that differ by hundreds between the halves."""
    d, dtype = 64, B.AD_BF16
    q, v = (quantize(SI.make_array(s, sd), dtype) for s, sd in (((bsz, l, heads * d), 81), ((bsz, lk, heads * d), 83)))
    k = SI.make_array((bsz, lk, heads * d), 82)
    k[..., ::d] += ramp * np.linspace(-8.0, 8.0, lk)[None, :, None]
    q[..., ::d] = quantize(np.abs(q[..., ::d]) * 4, dtype)
    k = quantize(k, dtype)
    got = run_attention(dtype, q, k, v, heads, True)
    assert_kernel_close(got, P.attention(mfma2_contract(q, d, -1, dtype, True, lk), k, v, heads), dtype, c=4.0)


@pytest.mark.parametrize("masked", [[(160, 300)], [(192, 299)], [(100, 224)], [(32, 200), (230, 290)]], ids=str)
def test_attention_keys_shared_out_scores_of_minus_infinity(masked):
    """The second group may have no finite score at first, or at all."""
    l, lk, d, dtype = 40, 300, 64, B.AD_BF16
    q, k, v = (quantize(SI.make_array((1, n, d), 86 + i), dtype) for i, n in enumerate((l, lk, lk)))
    q[..., 0], k[..., 0] = quantize(1e20, dtype), 0.0
    keep = np.ones(lk, bool)
    for a, b in masked:
        keep[a:b] = False
    k[:, ~keep, 0] = quantize(-1e20, dtype)
    got = run_attention(dtype, q, k, v, 1, True)
    qr = mfma2_contract(q, d, -1, dtype, True, lk)
    assert_kernel_close(got, P.attention(qr, k[:, keep], v[:, keep], 1), dtype, c=4.0)


# ---------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("batch", [1, 2])
def test_sampler_update(batch):
    T, n = 50, 4 * 24 * 24
    taus, acp = SM.timesteps(T), SM.alphas_cumprod()
    x = SI.make_array((n,), 81)
    eps = SI.make_array((batch, n), 82)
    for i, sampler in [(0, B.AD_DDIM), (17, B.AD_DDIM), (49, B.AD_DDIM), (3, B.AD_EULER)]:
        e = SM.cfg_combine(eps.astype(np.float64), 7.5)
        if sampler == B.AD_DDIM:
            ref = SM.ddim_step(x, e, i, taus, acp)
            a, a2 = acp[taus[i]], (acp[taus[i + 1]] if i + 1 < T else 1.0)
            cx, ce = math.sqrt(a2 / a), math.sqrt(1 - a2) - math.sqrt(a2) * math.sqrt(1 - a) / math.sqrt(a)
        else:
            ref = SM.euler_step(x, e, i, taus, acp)
            cx, ce = 1.0, SM.sigma(i + 1, taus, acp) - SM.sigma(i, taus, acp)
        dx, de = dev_f32(x), dev_f32(eps)
        B.check(lib.ad_sampler_update_raw(p(dx), p(de), n, batch, cx, ce, 7.5, stream_ptr()))
        sync()
        assert rel_l2(host(dx), ref) < 1e-6


@pytest.mark.parametrize("dtype", [B.AD_F32, B.AD_BF16])
@pytest.mark.parametrize("frames,positions,c,heads", [(16, 37, 320, 8), (3, 64, 64, 4), (16, 5, 1280, 8), (1, 9, 64, 8), (7, 130, 96, 2), (16, 33, 640, 8),
                                                      (5, 21, 60, 4), (13, 4097, 64, 1)])
def test_attention_over_frames(dtype, frames, positions, c, heads):
    """Temporal layer kernel: the sequences are the frames of each spatial position (row = frame * positions + p)."""
    rows = frames * positions
    ld = c + 8                                               # padded leading dimension
    q, k, v = (quantize(SI.make_array((rows, ld), 700 + i), dtype) for i in range(3))
    out = torch.full((rows, ld), float("nan"), device=DEV, dtype=tdtype(dtype))
    dq, dk, dv = dev(q, dtype), dev(k, dtype), dev(v, dtype)
    B.check(B.lib.ad_attention_frames_forward(dtype, p(dq), p(dk), p(dv), frames, positions, c, heads,
                                              ld, ld, ld, ld, p(out), stream_ptr()))
    torch.cuda.synchronize()
    seq = lambda a: a[:, :c].reshape(frames, positions, c).transpose(1, 0, 2)        # [positions][frames][c]
    ref = P.attention(seq(q), seq(k), seq(v), heads).transpose(1, 0, 2).reshape(rows, c)
    got = host(out)
    assert np.isnan(got[:, c:]).all()                        # nothing written past the row
    assert_kernel_close(got[:, :c], ref, dtype)


@pytest.mark.parametrize("rows,n_out,k,small", [
    (45, 64, 4800, True), (45, 64, 4832, False),          # tiles of 16x16: 150 k-tiles of 32 at the most
    (288, 256, 3200, True), (288, 256, 3232, False),      # 16x32: 100
    (512, 320, 2400, True), (512, 320, 2432, False),      # 32x32: 75
    (18, 260, 2304, True)])
def test_fp32_long_k_in_small_tiles(rows, n_out, k, small):
    """fp32 layers of few rows and a long K: small tiles up to 600 KiB a workgroup, K shared out over workgroups (which needs scratch) beyond."""
    x = SI.make_array((1, k, rows, 1), 321)
    w = SI.make_array((n_out, k, 1, 1), 322, k ** -0.5)
    bias, res = SI.make_array((n_out,), 323, 0.1), SI.make_array((1, rows, 1, n_out), 324)
    ref = P.conv2d(x, w, bias)
    got, _ = run_conv(B.AD_F32, x, None, w, bias, residual=res, splitk=True)
    assert (run_conv.last_ws_bytes == 0) == small
    assert_kernel_close(nhwc_to_nchw(got), ref + nhwc_to_nchw(res), B.AD_F32)


@pytest.mark.parametrize("rows,n_out,k", [(18, 256, 2304), (18, 256, 4608), (45, 64, 4800), (288, 256, 3200), (512, 320, 2400)])
def test_fp32_small_tiles_add_up_by_parts(rows, n_out, k):
    """A wavefront's sum goes to another one every 128 terms.  Error against 64 bits, 2-norm: 2.1e-7 at any K (a chain of 128 roundings that grow with it, eight wavefronts);
    in one chain a wavefront 3.1e-7 at K = 2304, 4.4e-7 at 4608 and 4800."""
    x = SI.make_array((1, k, rows, 1), 331).astype(np.float32)
    w = (SI.make_array((n_out, k, 1, 1), 332) * k ** -0.5).astype(np.float32)
    got, _ = run_conv(B.AD_F32, x, None, w, None, splitk=True)
    assert run_conv.last_ws_bytes == 0
    ref = P.conv2d(x.astype(np.float64), w.astype(np.float64), None)
    assert rel_l2(nhwc_to_nchw(got), ref) < 2.6e-7, rel_l2(nhwc_to_nchw(got), ref)

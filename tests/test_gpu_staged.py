"""The register-staged tiled kernel (float operands in three 16-bit parts, ragged channel counts, channels-first tensors)
against the oracle, over its gathers and tiles, and its answers for values that are not finite."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import oracle
from paper_2309_06626_amd import binding as B
from paper_2309_06626_amd import runtime as R
from parity import check_layer, rows_view
from test_gpu_compact import check_compact_output, run_compact_out
from test_gpu_parity import spec_of
from test_gpu_residual import check as check_residual

pytestmark = pytest.mark.gpu

TILES = ["128x64", "128x32", "64x64", "64x64x2", "64x128", "64x128x2", "64x32", "128x64x2", "64x32x4"]
CASES = [
    dict(n=2, cin=16, h=19, w=17, cout=160, k=3),                      # float: K tiles that span taps; two ragged channel tiles
    dict(n=2, cin=32, h=11, w=13, cout=33, k=3, s=2, sp=0.3),          # float: a K tile per tap; output rows at odd addresses
    dict(n=1, cin=13, h=12, w=10, cout=51, k=3, p=2, d=2, sp=0.4),     # ragged last group, dilation
    dict(n=3, cin=51, h=9, w=9, cout=102, k=1, p=0, sp=0.5),           # ragged pointwise
    dict(n=1, cin=9, h=15, w=11, cout=8, k=5, p=2, sp=0.0),            # one entry past a group; every row kept
    dict(n=2, cin=3, h=14, w=14, cout=24, k=8, s=2, p=3, sp=0.6),      # fewer channels than a group, the widest window
    dict(n=1, cin=72, h=3, w=2, cout=5, k=3, sp=0.5),                  # three rows
]


@pytest.mark.parametrize("tile", ["128x64", "128x64x2", "128x32", "128x32x2", "64x64", "64x64x2", "64x32", "64x32x2", "64x32x4"])
@pytest.mark.parametrize("cout", [84, 80])
@pytest.mark.parametrize("cin,k", [(32, 1), (64, 1), (96, 1), (4, 3), (32, 3), (64, 3), (40, 3), (32, 2)])
def test_float_walks(cin, k, cout, tile, monkeypatch):
    """One to eighteen K tiles, odd and even, tiles within a tap and across taps; shares that differ by a tile or hold none; the
    step past the end of a walk, whose operands nothing may use; rows of whole 16-channel blocks and of whole groups only."""
    monkeypatch.setenv("SPARSE_CONV_STAGE_TILE", tile)
    layer = check_layer(W.make_conv_inputs(spec_of(n=2, cin=cin, h=11, w=9, cout=cout, k=k, p=k // 2, dtype="f32", sp=0.35), 1571))
    for which in (0, 1):
        assert B.sparse_conv_plan_kernel(layer.plan, which) == "tile_staged"
        assert ["%d" % v for v in B.sparse_conv_plan_tiles(layer.plan, which)[:2]] == tile.split("x")[:2]


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("layout", ["nhwc", "nchw"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_gathers_and_tiles(case, layout, dtype, monkeypatch):
    spec = spec_of(dtype=dtype, layout=layout, **CASES[case])
    staged = dtype == "f32" or layout == "nchw" or spec.c_in % 8
    for tile in TILES:
        direct = dtype == "f32" and layout == "nhwc" and spec.c_in % 4 == 0 and spec.c_out % 4 == 0     # straight into LDS
        if not staged or (direct and tile.startswith("64x128")) or (tile not in TILES[:6] and not direct):
            continue
        monkeypatch.setenv("SPARSE_CONV_STAGE_TILE", tile)
        layer = check_layer(W.make_conv_inputs(spec, 1500 + case))
        if B.sparse_conv_plan_kernel(layer.plan, 0) == "band_row_segments" or "row_segments" in B.sparse_conv_plan_kernel(layer.plan, 0):
            return                                                     # (small-channel 16-bit stems have a kernel of their own)
        assert B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_staged"
        assert ["%d" % v for v in B.sparse_conv_plan_tiles(layer.plan, 0)[:2]] == tile.split("x")[:2]
    if staged:
        monkeypatch.delenv("SPARSE_CONV_STAGE_TILE")
        check_layer(W.make_conv_inputs(spec.with_(mask_mode="spatial"), 1520 + case), out_mode=B.SC_OUT_SCATTER_ONLY)


@pytest.mark.parametrize("dtype,cin,layout", [("f32", 32, "nhwc"), ("f32", 7, "nhwc"), ("bf16", 21, "nhwc"), ("f16", 16, "nchw")])
def test_shortcut_and_compact_rows(dtype, cin, layout):
    for cout in (16, 27):
        spec = spec_of(2, cin, 9, 12, cout, k=1, p=0, dtype=dtype, layout=layout, relu=False)
        check_residual(spec, 1540, True, want_kernel=("tile_staged",))
        if layout == "nhwc":
            check_residual(spec, 1541, False, y_compact=True)
            check_residual(spec, 1542, True, y_compact=True, x_compact=True)
            check_compact_output(spec.with_(kh=3, kw=3, pad_h=1, pad_w=1), 1543)


@pytest.mark.parametrize("sx,sw", [(2.0 ** -60, 2.0 ** -50), (2.0 ** 60, 2.0 ** 50), (2.0 ** -110, 2.0 ** 100)])
def test_float_parts_at_the_ends_of_the_range(sx, sw):
    spec = spec_of(1, 24, 10, 10, 36, dtype="f32", bias=False)          # (no band kernel: output channels off the 16-channel group)
    ci = W.make_conv_inputs(spec, 1560)
    ci.x, ci.w = ci.x * np.float32(sx), ci.w * np.float32(sw)
    assert B.sparse_conv_plan_kernel(check_layer(ci).plan, 0) == "tile_staged"


VALUES = [np.inf, -np.inf, np.nan, 3.4e38, -3.4028235e38]


@pytest.mark.parametrize("dtype,cin,layout", [("f32", 32, "nhwc"), ("f32", 13, "nhwc"), ("f32", 8, "nchw"), ("bf16", 13, "nhwc"),
                                              ("f16", 27, "nhwc"), ("bf16", 8, "nchw")])
@pytest.mark.parametrize("where", ["x", "w"])
def test_values_that_are_not_finite(dtype, cin, layout, where):
    """The same finite, infinite and not-a-number results as the kernel that gathers element by element or in 16-byte
    groups (a forced tile), which adds the plain products; what stays finite agrees with it."""
    for i, value in enumerate(VALUES):
        if abs(value) > 6e4 and np.isfinite(value) and dtype == "f16":
            continue
        spec = spec_of(1, cin, 9, 9, 40, dtype=dtype, layout=layout, relu=False, sp=0.2)
        ci = W.make_conv_inputs(spec, 1570 + i)
        x, w = ci.x.copy(), ci.w.copy()
        flat = (x if where == "x" else w).reshape(-1)
        with np.errstate(all="ignore"):
            flat[[flat.size // 2, flat.size - 1]] = W.quantize(np.array([value, value], np.float32), dtype) if np.isfinite(value) else value
        w.reshape(-1)[::7] = 0.5                    # filters whose later parts are zero
        layer = R.ConvLayer(spec, w, ci.bias, ci.mask)
        assert B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_staged"
        dev = R.to_device(x, dtype)
        a = layer.sparse(dev).float()
        B.sparse_conv_plan_set_tiles(layer.plan, 0, 64, 64)
        assert B.sparse_conv_plan_kernel(layer.plan, 0) != "tile_staged"
        b = layer.sparse(dev).float()
        torch.cuda.synchronize()
        assert torch.equal(a.isnan(), b.isnan()), (value, where)
        assert torch.equal(a.isinf(), b.isinf()) and torch.equal(a[a.isinf()], b[b.isinf()]), (value, where)
        fin = a.isfinite()
        tol = {"f32": 2e-5, "bf16": 2e-2, "f16": 4e-3}[dtype]
        assert torch.allclose(a[fin], b[fin], rtol=tol, atol=tol * float(b[fin].abs().max().clamp(max=100)))


# The kernel that goes straight into LDS, groups and ragged groups through registers, channels first; K in one and in two shares.
FLOAT_FORMS = [(32, 40, "nhwc", "64x32"), (32, 40, "nhwc", "64x64x2"), (20, 33, "nhwc", "64x64"), (13, 40, "nhwc", "64x64x2"), (8, 40, "nchw", "64x64")]


def float_form(form, monkeypatch, where=None, **kw):
    cin, cout, layout, tile = form
    monkeypatch.setenv("SPARSE_CONV_STAGE_TILE", tile)
    return spec_of(1, cin, 9, 10, cout, dtype="f32", layout=layout, relu=False, bias=False, sp=0.2, **kw)


# largest finite products whose leading parts multiply to infinity: a first part rounds up to 2^64
NEAR_THE_TOP = [2.0 ** 64 * (1 - 2.0 ** -24), 2.0 ** 64 * (1 - 2.0 ** -10)]


@pytest.mark.parametrize("value", NEAR_THE_TOP)
@pytest.mark.parametrize("form", FLOAT_FORMS)
def test_finite_products_of_values_that_round_up(form, value, monkeypatch):
    """x * w just below the largest float, one product a sum; and such a product beside one of the other sign."""
    spec = float_form(form, monkeypatch, k=1, p=0)
    ci = W.make_conv_inputs(spec, 1670)
    v = np.float32(value)
    x, w = np.zeros_like(ci.x), np.zeros_like(ci.w)
    ch = (slice(None), slice(None), slice(None)) if spec.layout == "nhwc" else ()
    x[(*ch, 2) if ch else (slice(None), 2)] = v
    x[(*ch, 7) if ch else (slice(None), 7)] = v
    wv = np.moveaxis(w, 3 if spec.layout == "nhwc" else 1, 0)          # [Cin, Cout, ...]
    wv[2] = v
    wv[7, ::2] = -v * np.float32(0.5)
    layer = R.ConvLayer(spec, w, ci.bias, ci.mask)
    assert B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_staged"
    y = rows_view(spec, R.to_host_f32(layer.sparse(R.to_device(x, "f32"))))[ci.mask == 1]
    top = float(v) * float(v)
    want = np.where(np.arange(spec.c_out) % 2 == 0, 0.5 * top, top)
    assert np.all(np.abs(y - want) <= 2.0 ** -22 * top)


@pytest.mark.parametrize("sx,sw", [(2.0 ** -118, 1.0), (1.0, 2.0 ** -118), (2.0 ** -124, 1.0), (1.0, 2.0 ** -124), (2.0 ** -126, 2.0 ** 100),
                                   (2.0 ** 100, 2.0 ** -126), (2.0 ** -60, 2.0 ** -50), (2.0 ** 60, 2.0 ** 50), (2.0 ** -110, 2.0 ** 100)])
@pytest.mark.parametrize("form", FLOAT_FORMS)
def test_small_and_large_operands_keep_all_their_bits(form, sx, sw, monkeypatch):
    spec = float_form(form, monkeypatch)
    ci = W.make_conv_inputs(spec, 1680)
    ci.x, ci.w = ci.x * np.float32(sx), ci.w * np.float32(sw)
    layer = check_layer(ci)
    assert B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_staged"


@pytest.mark.parametrize("sx,sg", [(2.0 ** -118, 1.0), (1.0, 2.0 ** -118), (2.0 ** -124, 2.0 ** 100), (2.0 ** 100, 2.0 ** -126), (2.0 ** 60, 2.0 ** 50)])
def test_float_filter_gradient_keeps_small_and_large_operands(sx, sg):
    spec, x, dy, kept, layer, bwd = filter_gradient_case(1690)
    x, dy = x * np.float32(sx), dy * np.float32(sg)
    got, want = filter_gradients(spec, x, dy, kept, bwd)
    assert np.linalg.norm(got - want) <= 2e-6 * np.linalg.norm(want)


@pytest.mark.parametrize("value", NEAR_THE_TOP)
def test_float_filter_gradient_of_values_that_round_up(value):
    """One product just below the largest float in a filter entry's sum."""
    spec, x, dy, kept, layer, bwd = filter_gradient_case(1691)
    x[:], dy[:] = 0.0, 0.0
    row = int(np.flatnonzero(kept)[40])
    n, oy, ox = row // 81, row % 81 // 9, row % 9
    x[n, oy, ox, 5], dy[n, oy, ox, 3] = value, -value
    got, want = filter_gradients(spec, x, dy, kept, bwd)
    assert np.isfinite(got).all() and np.all(np.abs(got - want) <= 2.0 ** -22 * value * value)


def filter_gradient_case(seed):
    spec = W.ConvSpec("wg", n=2, c_in=16, h=9, w=9, c_out=24, dtype="f32", sparsity=0.3, relu=False)
    ci = W.make_conv_inputs(spec, seed)
    dy = np.random.default_rng(seed).standard_normal(spec.y_shape()).astype(np.float32)
    layer = R.ConvLayer(spec, ci.w, ci.bias, ci.mask)
    return spec, ci.x.copy(), dy, ci.mask == 1, layer, B.sparse_conv_backward_plan(layer.plan, layer.w)


def filter_gradients(spec, x, dy, kept, bwd):
    dw = torch.empty(spec.w_shape(), dtype=torch.float32, device="cuda:0")
    B.sparse_conv_backward_run(bwd, R.to_device(x, "f32"), None, R.to_device(dy, "f32"), dw=dw)
    a = np.pad(x.astype(np.float64), ((0, 0), (1, 1), (1, 1), (0, 0)))
    a = np.stack([a[:, i:i + spec.h, j:j + spec.w] for i in range(3) for j in range(3)], 3).reshape(spec.m, -1)
    g = dy.astype(np.float64).reshape(spec.m, -1)
    return dw.cpu().numpy().astype(np.float64), (g[kept].T @ a[kept]).reshape(spec.w_shape())


@pytest.mark.parametrize("dtype,layout,case", [
    ("f32", "nhwc", dict(n=16, cin=64, h=12, w=12, cout=192)),          # staged, in one, two or four shares
    ("f32", "nhwc", dict(n=4, cin=16, h=56, w=56, cout=16)),            # around the line between band and staged
    ("f32", "nhwc", dict(n=2, cin=24, h=14, w=14, cout=35, k=1, p=0)),  # output rows off the 16-byte group
    ("f16", "nhwc", dict(n=8, cin=51, h=14, w=14, cout=102)),
    ("f32", "nchw", dict(n=2, cin=64, h=14, w=14, cout=64)),
])
def test_tuned_staged_layers(dtype, layout, case):
    """Whatever sparse_conv_plan_tune picks: the oracle's results, kept rows with the bits of the dense run, and the model's
    choice again after a new mask."""
    spec = spec_of(dtype=dtype, layout=layout, sp=0.5, **case)
    ci = W.make_conv_inputs(spec, 1595)
    layer = R.ConvLayer(spec, ci.w, ci.bias, ci.mask)
    x, y, d = R.to_device(ci.x, dtype), layer.new_output(), layer.new_output()
    state = lambda: [(B.sparse_conv_plan_kernel(layer.plan, i), B.sparse_conv_plan_tiles(layer.plan, i)) for i in (0, 1)]
    model = state()
    B.sparse_conv_plan_tune(layer.plan, x, layer.bias, y)
    assert state()[0][0] == state()[1][0] or "tile_masked_store" in state()[0][0]
    B.dense_conv_run(layer.plan, x, layer.bias, d)
    torch.cuda.synchronize()
    kept = ci.mask == 1
    got, ref = rows_view(spec, R.to_host_f32(y)), rows_view(spec, oracle.masked_conv2d(spec, ci.x, ci.w, ci.bias, ci.mask))
    assert np.linalg.norm(got - ref) <= {"f32": 1e-5, "f16": 4e-3}[dtype] * np.linalg.norm(ref)
    assert np.array_equal(rows_view(spec, R.bits_of(y))[kept], rows_view(spec, R.bits_of(d))[kept])
    assert (rows_view(spec, R.bits_of(y))[~kept] == 0).all()
    B.sparse_conv_plan_set_mask(layer.plan, torch.from_numpy(ci.mask).cuda())
    assert state() == model


def test_plan_refresh_reaches_the_staged_filters_and_tile():
    spec = spec_of(2, 40, 12, 12, 44, dtype="f32", sp=0.5)
    a, b = W.make_conv_inputs(spec, 1590), W.make_conv_inputs(spec, 1591)
    layer = R.ConvLayer(spec, a.w, b.bias, a.mask)
    assert B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_staged"
    layer.sparse(R.to_device(a.x, "f32"))
    B.sparse_conv_plan_set_filters(layer.plan, R.to_device(b.w, "f32"))
    B.sparse_conv_plan_set_mask(layer.plan, torch.from_numpy(b.mask).cuda())
    y = rows_view(spec, R.to_host_f32(layer.sparse(R.to_device(b.x, "f32"))))
    ref = rows_view(spec, oracle.masked_conv2d(spec, b.x, b.w, b.bias, b.mask))
    assert np.linalg.norm(y - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("shape", [
    dict(n=1, c_in=8, hw=5, c_out=8, k=1, sparsity=0.0),             # one ragged tile, fewer rows than a step
    dict(n=3, c_in=72, hw=17, c_out=136, k=3, sparsity=0.4),          # ragged tiles both ways, several splits, a ragged last step
    dict(n=2, c_in=24, hw=12, c_out=64, k=5, s=2, d=2, w=19, sparsity=0.7, mask_mode="spatial"),
    dict(n=1, c_in=16, hw=16, c_out=16, k=9, sparsity=0.5),           # a window past the validity bits: the float MFMA kernel
])
def test_float_filter_gradient(shape, monkeypatch):
    import test_gpu_backward as TB
    monkeypatch.setattr(TB, "TOL_F32_SUMS", 1e-5)
    TB.run_backward(TB.spec_of(dtype="f32", **shape), 1600)


@pytest.mark.parametrize("value", [np.inf, np.nan, 3.4e38])
def test_float_filter_gradient_of_values_that_are_not_finite(value):
    """dw has the finite, infinite and not-a-number entries of the plain sum over the kept rows."""
    spec = W.ConvSpec("wnf", n=2, c_in=16, h=9, w=9, c_out=24, dtype="f32", sparsity=0.3, relu=False)
    ci = W.make_conv_inputs(spec, 1620)
    x = ci.x.copy()
    x[0, 4, 4, 3] = x[1, 2, 7, 0] = value
    dy = np.random.default_rng(1621).standard_normal(spec.y_shape()).astype(np.float32)
    dy.reshape(-1)[::5] = 0.0
    layer = R.ConvLayer(spec, ci.w, ci.bias, ci.mask)
    bwd = B.sparse_conv_backward_plan(layer.plan, layer.w)
    dw = torch.empty(spec.w_shape(), dtype=torch.float32, device="cuda:0")
    B.sparse_conv_backward_run(bwd, R.to_device(x, "f32"), None, R.to_device(dy, "f32"), dw=dw)
    cols = torch.nn.functional.unfold(torch.from_numpy(x).permute(0, 3, 1, 2), 3, padding=1)        # [N, C * 9, L]
    a = cols.view(2, 16, 9, 81).permute(0, 3, 2, 1).reshape(162, 144)
    kept = torch.from_numpy(ci.mask).bool()
    want = (torch.from_numpy(dy).reshape(162, 24)[kept].t() @ a[kept]).view(24, 3, 3, 16)
    got = dw.cpu()
    assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf())
    fin = want.isfinite()
    assert torch.allclose(got[fin], want[fin], rtol=1e-4, atol=1e-4)


@pytest.mark.parametrize("dtype,staged", [("f32", False), ("f32", True), ("bf16", False), ("f16", False)])
@pytest.mark.parametrize("cin,cout,k", [(8, 40, 3), (64, 264, 1), (72, 16, 5)])
def test_refreshed_filters_equal_those_of_a_new_plan(cin, cout, k, dtype, staged, monkeypatch):
    """Forward and input gradient after set_filters (one launch each, the rotation folded in): the bits of fresh plans.
    staged: these layers are small enough for other kernels, so the float parts have to be asked for."""
    if staged:
        monkeypatch.setenv("SPARSE_CONV_STAGE_TILE", "64x32")
    spec = spec_of(2, cin, 9, 11, cout, k=k, p=k // 2, dtype=dtype, relu=False)
    a, b = W.make_conv_inputs(spec, 1630), W.make_conv_inputs(spec, 1631)
    x, dy = R.to_device(b.x, dtype), torch.randn(spec.y_shape(), device="cuda:0").to(B.TORCH_DTYPE[dtype])
    got = []
    for first in (a.w, b.w):
        layer = R.ConvLayer(spec, first, b.bias, b.mask)
        bwd = B.sparse_conv_backward_plan(layer.plan, layer.w)
        assert not staged or B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_staged"
        if first is a.w:
            w = R.to_device(b.w, dtype)
            B.sparse_conv_plan_set_filters(layer.plan, w)
            B.sparse_conv_backward_set_filters(bwd, w)
        y, dx = layer.sparse(x), torch.empty_like(x)
        B.sparse_conv_plan_set_tiles(layer.plan, 0, 64, 64)          # and the layout of the other kernels
        y2 = layer.sparse(x)
        B.sparse_conv_backward_run(bwd, x, y, dy, dx=dx)
        got.append([R.bits_of(t) for t in (y, y2, dx)])
    for p, q in zip(*got):
        assert np.array_equal(p, q)


@pytest.mark.parametrize("case", [
    dict(n=1, cin=16, h=16, w=16, cout=16),                          # unrolled window, one filter block
    dict(n=3, cin=32, h=5, w=32, cout=48, sp=0.3),                   # a full 32-row block, two filter blocks
    dict(n=2, cin=8, h=9, w=7, cout=80, k=3, s=2, p=1, sp=0.6),      # run-time window, four filter blocks
    dict(n=1, cin=16, h=8, w=11, cout=16, k=3, p=2, d=2, sp=0.95),   # bands without a kept row
])
@pytest.mark.parametrize("mask_mode", ["row", "spatial"])
def test_small_float_bands_share_the_window(case, mask_mode):
    spec = spec_of(dtype="f32", mask_mode=mask_mode, **case)
    for out_mode in (B.SC_OUT_ZERO_FILL, B.SC_OUT_SCATTER_ONLY):
        layer = check_layer(W.make_conv_inputs(spec, 1640), tiles=(-1, 0), out_mode=out_mode)
        assert B.sparse_conv_plan_kernel(layer.plan, 0) == "band"


@pytest.mark.parametrize("dtype,cin,layout", [("f32", 13, "nhwc"), ("bf16", 21, "nhwc"), ("f16", 16, "nchw"), ("f32", 16, "nchw")])
def test_layers_ignore_options_of_other_kernels(dtype, cin, layout):
    """The gather pipeline of 16-byte groups, and masked stores of NHWC runs, leave the other layers where they are."""
    spec = spec_of(1, cin, 9, 9, 24, dtype=dtype, layout=layout)
    options = [(B.SC_OPT_GATHER_PIPELINE, 1), (B.SC_OPT_GATHER_PIPELINE, 2)] + ([(B.SC_OPT_MASKED_STORE, 2)] if layout == "nchw" else [])
    for option, value in options:
        layer = check_layer(W.make_conv_inputs(spec, 1648), options={option: value})
        assert B.sparse_conv_plan_kernel(layer.plan, 0) == B.sparse_conv_plan_kernel(layer.plan, 1) == "tile_staged"


@pytest.mark.parametrize("case", [
    dict(n=4, cin=256, h=28, w=28, cout=256, k=1, p=0, dtype="f32"),                     # straight into LDS
    dict(n=16, cin=8, h=28, w=28, cout=256, k=1, p=0, dtype="f32", layout="nchw"),       # through registers, one K tile
    dict(n=1, cin=13, h=30, w=20, cout=160, k=3, dtype="bf16"),
])
def test_groups_of_both_runs(case):
    """The shares of K are chosen for the sparse and the dense run together: the same bits, and no dense run of several rounds of
    workgroups that fill a compute unit each."""
    spec = spec_of(sp=0.5, relu=False, **case)
    layer = check_layer(W.make_conv_inputs(spec, 1649), sample_rows=300)
    assert B.sparse_conv_plan_kernel(layer.plan, 0) == B.sparse_conv_plan_kernel(layer.plan, 1) == "tile_staged"
    ci = W.make_conv_inputs(spec, 1649)
    x, y, d = R.to_device(ci.x, spec.dtype), layer.new_output(), layer.new_output()
    layer.sparse(x, y)
    B.dense_conv_run(layer.plan, x, layer.bias, d)
    assert np.array_equal(rows_view(spec, R.bits_of(y))[ci.mask == 1], rows_view(spec, R.bits_of(d))[ci.mask == 1])
    if spec.c_in == 256:                               # four shares of 64 x 32 tiles took the dense run 12.7 us in two rounds, 9.0 now
        bm, bn, wgs = B.sparse_conv_plan_tiles(layer.plan, 1)
        assert wgs <= 256 or (bm, bn) != (64, 32)


@pytest.mark.parametrize("cin,k", [(32, 1), (8, 1), (128, 1), (4, 3)])
def test_short_float_walks_stay_with_the_float_tiles(cin, k):
    """Plain and compact runs of small float layers of at most four K tiles; fused ones, and a fifth tile, are staged."""
    spec = spec_of(2, cin, 19, 13, 48, k=k, p=k // 2, dtype="f32", relu=False)
    layer = check_layer(W.make_conv_inputs(spec, 1651))
    assert "staged" not in B.sparse_conv_plan_kernel(layer.plan, 0) and "staged" not in B.sparse_conv_plan_kernel(layer.plan, 1)
    assert B.sparse_conv_plan_fused_kernel(layer.plan, 0) == "tile_staged"
    check_compact_output(spec, 1652)
    check_residual(spec, 1653, True, want_kernel=("tile_staged",))
    longer = check_layer(W.make_conv_inputs(spec.with_(c_in=160), 1654))
    assert B.sparse_conv_plan_kernel(longer.plan, 0) == "tile_staged"


@pytest.mark.parametrize("dtype,sp,kernel", [("bf16", 0.1, "tile_elements"), ("f32", 0.1, "tile_elements"), ("bf16", 0.5, "tile_staged"), ("f32", 0.5, "tile_staged")])
def test_many_outputs_behind_one_ragged_k_tile(dtype, sp, kernel):
    spec = spec_of(4, 13, 56, 56, 256, k=1, p=0, dtype=dtype, sp=sp)
    layer = check_layer(W.make_conv_inputs(spec, 1655), sample_rows=300)
    assert B.sparse_conv_plan_kernel(layer.plan, 0) == B.sparse_conv_plan_kernel(layer.plan, 1) == kernel


def test_small_float_layers_without_a_band_form_run_staged(monkeypatch):
    """Small float layers keep the band kernel; their fused and compact runs, which it does not have, take the staged one."""
    spec = spec_of(2, 16, 12, 11, 16, dtype="f32", relu=False)
    layer, ci = check_compact_output(spec, 1645)
    assert B.sparse_conv_plan_kernel(layer.plan, 0) == "band"
    assert B.sparse_conv_plan_fused_kernel(layer.plan, 0) == B.sparse_conv_plan_fused_kernel(layer.plan, 1) == "tile_staged"
    check_residual(spec, 1646, True)
    check_residual(spec, 1647, False, y_compact=True)
    x = R.to_device(ci.x, "f32")
    _, bits = run_compact_out(layer, x)
    same = []
    for tile in ("64x32", "64x32x2", "64x32x4"):                       # (results depend on the shares of K, not on the tile)
        monkeypatch.setenv("SPARSE_CONV_STAGE_TILE", tile)
        same.append(np.array_equal(run_compact_out(R.ConvLayer(spec, ci.w, ci.bias, ci.mask), x)[1], bits))
    assert any(same)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("case", [
    dict(n=2, cin=64, h=15, w=13, cout=80, sp=0.4),                   # nine K tiles: shares of five and four
    dict(n=1, cin=128, h=9, w=20, cout=64, k=3, s=2, sp=0.0),          # every row kept
    dict(n=1, cin=64, h=7, w=7, cout=160, k=5, p=2, sp=0.9),           # five kept rows, ragged channel tile
])
def test_groups_of_wavefronts_share_k(case, dtype, monkeypatch):
    """Two groups of wavefronts of the buffer-load kernel: against the oracle, compact rows and shortcut sums included."""
    monkeypatch.setenv("SPARSE_CONV_TILE_GROUPS", "64x64x2")
    monkeypatch.setenv("SPARSE_CONV_BAND_KERNEL", "single")
    spec = spec_of(dtype=dtype, **case)
    for out_mode in (B.SC_OUT_ZERO_FILL, B.SC_OUT_SCATTER_ONLY):
        layer = check_layer(W.make_conv_inputs(spec, 1650), out_mode=out_mode)
        assert B.sparse_conv_plan_tiles(layer.plan, 0)[:2] == (64, 64)
    check_residual(spec.with_(relu=False), 1651, True, want_kernel=("tile_lds_direct",))
    if spec.sparsity > 0:
        check_compact_output(spec, 1652)


@pytest.mark.parametrize("dtype,shape", [
    ("bf16", dict(n=64, cin=512, h=7, w=7, cout=512)),                  # in the place of a split into four
    ("f16", dict(n=30, cin=384, h=13, w=13, cout=384)),
    ("bf16", dict(n=2, cin=256, h=40, w=40, cout=256)),
    ("bf16", dict(n=12, cin=320, h=14, w=14, cout=448, k=5, p=2)),
    ("f16", dict(n=64, cin=256, h=14, w=14, cout=512, s=2)),
])
def test_automatic_groups_add_in_the_order_of_the_split_they_replace(dtype, shape, monkeypatch):
    """Results do not depend on whether two groups of wavefronts or the split-K launch contracts a layer: the same bits."""
    monkeypatch.setenv("SPARSE_CONV_WINDOW_TILE", "0x0")               # (most of these layers are the window kernel's otherwise)
    spec = spec_of(dtype=dtype, sp=0.5, **shape)
    ci = W.make_conv_inputs(spec, 1660)
    layer = R.ConvLayer(spec, ci.w, ci.bias, ci.mask)
    x = R.to_device(ci.x, dtype)
    got = []
    for stream_k in (0, 8):                                            # (any such request keeps the groups out)
        B.sparse_conv_plan_set_option(layer.plan, B.SC_OPT_STREAM_K, stream_k)
        got.append((B.sparse_conv_plan_kernel(layer.plan, 0), B.sparse_conv_plan_tiles(layer.plan, 0), R.bits_of(layer.sparse(x))))
    if got[1][0] == "tile_stream_k":                                   # (no split here: no groups either)
        B.sparse_conv_plan_set_option(layer.plan, B.SC_OPT_STREAM_K, 1)
        got[1] = (B.sparse_conv_plan_kernel(layer.plan, 0), B.sparse_conv_plan_tiles(layer.plan, 0), R.bits_of(layer.sparse(x)))
        assert got[0][:2] == got[1][:2]
    elif got[0][0] == "tile_lds_direct":
        assert got[1][0] == "tile_split_k"
    assert np.array_equal(got[0][2], got[1][2])
    if shape["cin"] == 512:
        assert got[0][0] == "tile_lds_direct" and got[0][1][:2] == (64, 64) and got[1][0] == "tile_split_k"

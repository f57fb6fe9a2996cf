"""Window kernel (3x3 and 5x5 layers at stride 1 whose channels are whole 16-byte groups: every input pixel of a tile once in LDS, filters straight
into registers) against the oracle, through the C ABI."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as W
from oracle import oracle
from paper_2309_06626_amd import binding as B
from paper_2309_06626_amd import runtime as R
from parity import TOL, assert_close, check_layer, row_mask, rows_view
from test_gpu_compact import check_compact_output
from test_gpu_parity import spec_of
from test_gpu_residual import check as check_residual
from test_gpu_slab import slab_fits

pytestmark = pytest.mark.gpu

TILES = [(256, 128), (128, 128), (128, 64), (64, 128), (64, 64)]
SHAPES = {
    "one_chunk_edge_channels": dict(n=2, cin=64, h=15, w=13, cout=80),             # no second slab; half a block of channels
    "images_in_a_tile": dict(n=9, cin=128, h=7, w=5, cout=144, sp=0.3),            # maps smaller than a set of lanes
    "no_padding": dict(n=2, cin=128, h=12, w=10, cout=320, p=0),
    "padding_2": dict(n=1, cin=192, h=8, w=30, cout=16, p=2, sp=0.0),              # output larger than the input, every row kept
    "one_row_kept": dict(n=1, cin=64, h=6, w=6, cout=32, sp=0.97),
    "last_chunk_of_8": dict(n=2, cin=72, h=9, w=11, cout=24),                       # half a K step behind the first chunk; half a block
    "last_chunk_of_40": dict(n=3, cin=104, h=10, w=7, cout=104, sp=0.3),
    "under_a_chunk": dict(n=2, cin=24, h=11, w=12, cout=152, sp=0.2),
    "window_5x5": dict(n=3, cin=80, h=9, w=11, cout=72, k=5, p=2),
    "window_5x5_no_padding": dict(n=2, cin=136, h=12, w=9, cout=96, k=5, p=0, sp=0.3),
    "wide_map_most_kept": dict(n=2, cin=64, h=9, w=60, cout=64, sp=0.3),            # five to seven rows of 62 pixels
    "wide_map": dict(n=1, cin=64, h=4, w=120, cout=64, sp=0.7),                    # a tap row is most of the slab
}


def fits(spec, mask, tile):
    """Whether the widest slab of a tile fits: at most 512 pixels, and its one or two buffers beside the rest of LDS."""
    rows = oracle.compact_rows(row_mask(spec, mask))
    hp, wp = spec.h + 2 * spec.pad_h, spec.w + 2 * spec.pad_w
    span = 0
    for r in (rows, np.arange(spec.m)) if rows.size == spec.m else (rows,):
        vrow = (r // (spec.ho * spec.wo)) * hp + (r % (spec.ho * spec.wo)) // spec.wo
        bm = tile[0]
        first, last = vrow[::bm], vrow[np.minimum(np.arange(0, r.size, bm) + bm, r.size) - 1]
        span = max(span, int((last + spec.kh - first).max()))
    slab = -(-span * wp * 144 // 8192) * 8192 * (2 if spec.c_in > 64 else 1)
    sums = {(256, 128): 0, (128, 128): 4, (128, 64): 4, (64, 128): 2, (64, 64): 2}[tile] * 32768
    rest = tile[0] * 12 + tile[1] * 4 + 2048 + 128 + (tile[0] + 64) * 4
    return span * wp <= 512 and max(slab, sums) + rest <= 160 * 1024


def assert_window(layer, spec, mask, tile):
    """Wherever the tile's slabs fit, the plain and the fused sparse and dense runs are the window kernel's in that tile; elsewhere none is."""
    for which, m in ((0, mask), (1, np.ones_like(mask))):
        took = B.sparse_conv_plan_kernel(layer.plan, which) == "tile_window"
        assert took == (B.sparse_conv_plan_fused_kernel(layer.plan, which) == "tile_window") == fits(spec, m, tile)
        assert not took or B.sparse_conv_plan_tiles(layer.plan, which)[:2] == tile
    return layer


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("shape", list(SHAPES))
def test_window_kernel_matches_the_oracle(shape, tile, dtype, monkeypatch):
    monkeypatch.setenv("SPARSE_CONV_WINDOW_TILE", "%dx%d" % tile)
    spec = spec_of(dtype=dtype, **SHAPES[shape])
    ci = W.make_conv_inputs(spec, 3000 + len(shape))
    assert_window(check_layer(ci), spec, ci.mask, tile)
    assert tile[0] > 64 or fits(spec, np.ones_like(ci.mask), tile)      # (something does run)


@pytest.mark.parametrize("cin,cout", [(128, 96), (88, 56)])
@pytest.mark.parametrize("tile", TILES)
def test_window_kernel_other_operands(tile, cin, cout, monkeypatch):
    """Rows left alone, compact rows, shortcut sums, a shared mask; masks with long runs of dropped rows; new masks."""
    monkeypatch.setenv("SPARSE_CONV_WINDOW_TILE", "%dx%d" % tile)
    spec = spec_of(3, cin, 10, 9, cout, sp=0.4)
    for seed, sp, out_mode in ((3100, spec, B.SC_OUT_SCATTER_ONLY), (3101, spec.with_(mask_mode="spatial"), B.SC_OUT_ZERO_FILL)):
        ci = W.make_conv_inputs(sp, seed)
        assert_window(check_layer(ci, out_mode=out_mode), sp, ci.mask, tile)
    assert_window(check_compact_output(spec, 3102)[0], spec, W.make_conv_inputs(spec, 3102).mask, tile)
    for sp in (0.4, 0.0, 0.9):                       # (at 0.9 most dropped rows lie behind the listed ones)
        s = spec.with_(sparsity=sp, relu=False)
        assert_window(check_residual(s, 3103, True), s, W.make_conv_inputs(s, 3103).mask, tile)
    s = spec.with_(sparsity=0.5)
    ci = W.make_conv_inputs(s, 3104)
    half = np.zeros_like(ci.mask)
    half[::2] = 1                                    # every other pixel: all rows of a set of lanes in half of the bank groups
    runs = np.sort(ci.mask)                          # all dropped rows in front
    for mask in (half, runs, runs[::-1].copy()):
        assert_window(check_layer(dataclasses.replace(ci, mask=mask)), s, mask, tile)
    layer = R.ConvLayer(s, ci.w, ci.bias, ci.mask)
    x = R.to_device(ci.x, spec.dtype)
    for mask in (runs, half):
        B.sparse_conv_plan_set_mask(layer.plan, torch.from_numpy(mask.astype(np.uint8)).cuda())
        fresh = R.ConvLayer(s, ci.w, ci.bias, mask)
        assert np.array_equal(R.bits_of(layer.sparse(x)), R.bits_of(assert_window(fresh, s, mask, tile).sparse(x)))
        assert_window(layer, s, mask, tile)


def test_values_outside_a_window_do_not_enter(monkeypatch):
    """Infinities of a pixel reach the rows whose window holds it and no others, at the borders of images too."""
    monkeypatch.setenv("SPARSE_CONV_WINDOW_TILE", "64x64")
    spec = spec_of(2, 64, 9, 8, 32, sp=0.0, relu=False)
    ci = W.make_conv_inputs(spec, 3200)
    layer = assert_window(R.ConvLayer(spec, ci.w, ci.bias, ci.mask), spec, ci.mask, (64, 64))
    assert B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_window"
    clean = layer.sparse(R.to_device(ci.x, spec.dtype)).clone()
    for n, y, x in ((0, 8, 7), (1, 0, 0), (0, 4, 0)):
        bad = ci.x.copy()
        bad[n, y, x, :] = np.inf
        got = layer.sparse(R.to_device(bad, spec.dtype))
        reached = torch.zeros(got.shape[:3], dtype=torch.bool, device=got.device)
        reached[n, max(y - 1, 0): y + 2, max(x - 1, 0): x + 2] = True
        assert torch.equal(got[~reached], clean[~reached]) and not torch.isfinite(got[reached].float()).any()


def test_refreshed_filters_reach_the_window_kernel(monkeypatch):
    monkeypatch.setenv("SPARSE_CONV_WINDOW_TILE", "64x128")
    spec = spec_of(2, 136, 9, 8, 72, sp=0.3)
    one, two = W.make_conv_inputs(spec, 3300), W.make_conv_inputs(spec, 3301)
    layer = assert_window(R.ConvLayer(spec, one.w, one.bias, one.mask), spec, one.mask, (64, 128))
    assert B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_window"
    fresh = R.ConvLayer(spec, two.w, one.bias, one.mask)
    B.sparse_conv_plan_set_filters(layer.plan, R.to_device(two.w, spec.dtype))
    x = R.to_device(one.x, spec.dtype)
    assert np.array_equal(R.bits_of(layer.sparse(x)), R.bits_of(fresh.sparse(x)))


def masks_for_spans(rng, length):
    """Kept rows that end early, begin late, lie in clumps or far apart, and stand around multiples of 1 024, where a workgroup's
    share of the row list ends."""
    half = (rng.random(length) < 0.5).astype(np.uint8)
    for lo, hi in ((0, length // 2), (0, 700), (length // 2, length), (length // 3, length // 2)):
        m = np.zeros_like(half)
        m[lo:hi] = half[lo:hi]
        yield m
    yield ((rng.random(length) < 0.9) & (np.arange(length) < length * 2 // 3)).astype(np.uint8)
    yield ((np.arange(length) // 300) % 2 == 0).astype(np.uint8)
    yield (np.abs((np.arange(length) + 512) % 1024 - 512) < 40).astype(np.uint8)
    yield (rng.random(length) < 0.02).astype(np.uint8)
    m = np.zeros_like(half)
    m[[0, 1, length - 1]] = 1
    yield m


@pytest.mark.parametrize("n,h,w,mode", [
    (1, 56, 56, "row"),                # four shares of the list
    (7, 23, 25, "row"), (5, 31, 11, "spatial"), (60, 9, 8, "row"),      # images across shares
    (1, 6800, 20, "row"),              # past 2^17 rows: the tables of several launches
])
def test_spans_of_tiles_across_the_shares_of_the_row_list(n, h, w, mode, monkeypatch):
    """The window and the slab kernel run exactly where the widest slab of their tiles fits."""
    rng = np.random.default_rng(n + h)
    spec = spec_of(n, 64, h, w, 128, mask_mode=mode, sp=0.5)
    masks = list(masks_for_spans(rng, spec.mask_len))
    took = 0
    for tile in ((64, 64), (128, 64), (256, 128)):
        monkeypatch.setenv("SPARSE_CONV_WINDOW_TILE", "%dx%d" % tile)
        layer = R.ConvLayer(spec, np.zeros((128, 3, 3, 64), np.float32), np.zeros(128, np.float32), masks[0], check_count=False)
        for mask in masks:
            B.sparse_conv_plan_set_mask(layer.plan, torch.from_numpy(mask).cuda())
            got = B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_window"
            assert got == fits(spec, mask, tile)
            took += got
            if tile[0] >= 128:
                B.sparse_conv_plan_set_option(layer.plan, B.SC_OPT_SLAB, tile[0])
                assert (B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_slab") == slab_fits(spec, mask, tile[0])
                B.sparse_conv_plan_set_option(layer.plan, B.SC_OPT_SLAB, 0)
    assert 0 < took < 3 * len(masks)


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("n,h,w,cout,sp,mode", [
    (13, 23, 25, 96, 0.4, "row"),                  # tiles across the shares of the row list
    (13, 23, 25, 104, 0.1, "spatial"),             # of 256 rows too
    (1, 6800, 20, 16, 0.1, "row"),                 # past 2^17 rows; more workgroups than compute units in every tile
])
def test_window_kernel_on_many_rows(n, h, w, cout, sp, mode, tile, monkeypatch):
    monkeypatch.setenv("SPARSE_CONV_WINDOW_TILE", "%dx%d" % tile)
    spec = spec_of(n, 80, h, w, cout, sp=sp, mask_mode=mode)
    ci = W.make_conv_inputs(spec, 3400)
    layer = assert_window(check_layer(ci, sample_rows=300), spec, ci.mask, tile)
    assert B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_window" or (tile[0] == 256 and sp == 0.4)


def clumped_masks(m):
    """Kept rows in a clump at either end or in the middle, or all but every 97th.  Of the tiles' shares of the map some hold no dropped row, some
    more than a list takes, some are longer than the 1 024 rows that are looked through for the list, with a full list and (the third) without."""
    for lo, hi in ((0, 40), (m // 3, m // 3 + 22), (0, m * 119 // 1000), (0, m // 2), (m // 2, m)):
        mask = np.zeros(m, np.uint8)
        mask[lo:hi] = 1
        yield mask
    yield (np.arange(m) % 97 != 0).astype(np.uint8)


@pytest.mark.parametrize("mode", ["row", "spatial"])
@pytest.mark.parametrize("tile", TILES)
def test_zeros_of_long_runs_of_dropped_rows(tile, mode, monkeypatch):
    """Every dropped row gets its zeros, or the shortcut alone, once and whoever writes it; kept rows keep their sums."""
    monkeypatch.setenv("SPARSE_CONV_WINDOW_TILE", "%dx%d" % tile)
    spec = spec_of(*((13, 80, 23, 25) if mode == "row" else (40, 80, 9, 9)), 104, sp=0.5, relu=False, mask_mode=mode)
    ci = W.make_conv_inputs(spec, 3600)
    x, res, took = R.to_device(ci.x, spec.dtype), None, 0
    for mask in clumped_masks(ci.mask.size):
        layer = assert_window(R.ConvLayer(spec, ci.w, ci.bias, mask, check_count=False), spec, mask, tile)
        took += B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_window"
        kept = torch.from_numpy(row_mask(spec, mask)).cuda().reshape(spec.n, spec.ho, spec.wo, 1).bool()
        res = torch.randn(spec.n, spec.ho, spec.wo, spec.c_out, device="cuda").bfloat16() if res is None else res
        plain, dense = layer.sparse(x, layer.new_output(fill_nan=True)), layer.dense(x)
        assert torch.equal(plain, torch.where(kept, plain, torch.zeros_like(plain)))
        assert_close(R.to_host_f32(plain * kept), R.to_host_f32(dense * kept), R.to_host_f32(dense.abs() * kept) + 0.1, TOL["bf16"], "kept rows")
        fused = B.sparse_conv_run_residual(layer.plan, x, layer.bias, res, layer.new_output(fill_nan=True))
        assert torch.equal(torch.where(kept, torch.zeros_like(fused), fused), torch.where(kept, torch.zeros_like(res), res))
        want = (plain.float() + res.float()) * kept
        assert_close(R.to_host_f32(fused * kept), want.cpu().numpy(), (plain.float().abs() + res.float().abs()).cpu().numpy() + 0.1, TOL["bf16"], "sums")
    assert took >= 3 or (mode == "spatial" and tile[0] > 64)


def test_zeros_of_a_dropped_half_are_shared_out():
    """A map whose lower half is dropped takes no longer than one of which every other row is (one workgroup wrote all those zeros: 30 us / 8)."""
    spec = spec_of(38, 160, 21, 19, 64, sp=0.5)
    ci = W.make_conv_inputs(spec, 3601)
    x, us = R.to_device(ci.x, spec.dtype), []
    for mask in (np.arange(spec.m) % 2 == 0, np.arange(spec.m) < spec.m // 2):
        layer = R.ConvLayer(spec, ci.w, ci.bias, mask.astype(np.uint8), check_count=False)
        assert B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_window"
        call, times = B.prepared_run(layer.plan, x, layer.bias, layer.new_output()), []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(40):
                call()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b) * 25)
        us.append(min(times))
    assert us[1] < 1.5 * us[0], us


@pytest.mark.parametrize("n,cin,h,w,cout,sp,want", [
    (62, 64, 53, 53, 32, 0.3, ("band", "band")),                     # us, band / cheapest other launch: 15.2 / 16.4, every row 13.9 / 21.0
    (33, 64, 69, 69, 16, 0.5, ("band", "band")),                     # 11.0 / 14.4, 12.3 / 20
    (58, 128, 31, 36, 16, 0.5, ("tile_window", "tile_lds_direct")),  # every row 41.9 / 12.0
    (2, 48, 48, 53, 32, 0.5, ("tile_window",) * 2),                  # every row 7.0 / 5.5
    (10, 32, 79, 77, 256, 0.5, ("band", "band")),                    # few channels, many outputs: several rounds of the window kernel
    (54, 32, 25, 23, 416, 0.5, ("tile_window",) * 2),                # 25.7 / 17.3, 31.4 / 20.2
    (48, 64, 55, 55, 16, 0.7, ("band", "band")),                     # 8.5 / 9.1
    (56, 64, 45, 45, 64, 0.25, ("band", "band")),                    # 16.4 / 19.1
])
def test_plain_band_kernel_gives_way_where_it_is_dearer(n, cin, h, w, cout, sp, want):
    spec = spec_of(n, cin, h, w, cout, sp=sp)
    mask = (np.random.default_rng(5).permutation(spec.m) >= round(sp * spec.m)).astype(np.uint8)
    layer = R.ConvLayer(spec, np.zeros((cout, 3, 3, cin), np.float32), np.zeros(cout, np.float32), mask, check_count=False)
    assert tuple(B.sparse_conv_plan_kernel(layer.plan, which) for which in (0, 1)) == want


@pytest.mark.parametrize("case,before,after", [
    (dict(n=17, cin=32, h=16, w=17, cout=16, k=5, p=2, sp=0.5), "band", "tile_window"),      # every row 10.3 us / 5.7
    (dict(n=62, cin=64, h=53, w=53, cout=32, sp=0.3), "band", "band"),                       # 13.9 / 31, in other tiles 21
    (dict(n=4, cin=64, h=56, w=56, cout=64, sp=0.5), "band_tap", "band_tap"),
])
def test_tuning_times_the_window_kernel_and_the_band_kernels(case, before, after):
    spec = spec_of(dtype="bf16", **case)
    ci = W.make_conv_inputs(spec, 3500)
    layer = R.ConvLayer(spec, ci.w, ci.bias, ci.mask)
    x, y = R.to_device(ci.x, spec.dtype), layer.new_output()
    assert B.sparse_conv_plan_kernel(layer.plan, 1) == before
    B.sparse_conv_plan_tune(layer.plan, x, layer.bias, y)
    assert B.sparse_conv_plan_kernel(layer.plan, 1) == after
    if after == "tile_window":                                          # (11.0 us / 6.4; its spans are worked out by the tuning)
        assert B.sparse_conv_plan_kernel(layer.plan, 0) == after
        assert np.array_equal(R.bits_of(layer.sparse(x))[ci.mask.reshape(spec.n, spec.ho, spec.wo) == 0], np.zeros((int((ci.mask == 0).sum()), spec.c_out), np.uint16))
    rows = np.unique(np.random.default_rng(5).integers(0, spec.m, 300)).astype(np.int64)
    ref, absum = oracle.masked_conv2d_rows(spec, ci.x, ci.w, ci.bias, np.ones_like(ci.mask), rows, want_absum=True)
    assert_close(rows_view(spec, R.to_host_f32(layer.dense(x)))[rows], ref, absum, TOL["bf16"], "tuned")
    B.sparse_conv_plan_set_mask(layer.plan, torch.from_numpy(ci.mask).cuda())
    assert B.sparse_conv_plan_kernel(layer.plan, 1) == after            # (a new mask leaves the dense run's choice)


def test_tuning_leaves_a_window_tile_that_was_asked_for(monkeypatch):
    for tile in ("64x64", "0x0"):
        monkeypatch.setenv("SPARSE_CONV_WINDOW_TILE", tile)
        spec = spec_of(17, 32, 16, 17, 16, k=5, p=2)
        ci = W.make_conv_inputs(spec, 3501)
        layer = R.ConvLayer(spec, ci.w, ci.bias, ci.mask)
        B.sparse_conv_plan_tune(layer.plan, R.to_device(ci.x, spec.dtype), layer.bias, layer.new_output())
        assert all((B.sparse_conv_plan_kernel(layer.plan, which) == "tile_window") == (tile == "64x64") for which in (0, 1))


@pytest.mark.parametrize("n,cin,h,w,cout,want", [
    (57, 48, 23, 26, 40, "tile_registers"),                          # every row, us, other tiles / this kernel: 9.3 / 10.4
    (37, 72, 31, 31, 40, "tile_registers"),                          # 12.0 / 13.1
    (60, 72, 45, 48, 40, "tile_window"),                             # 29.0 / 26.1
    (20, 64, 22, 22, 320, "tile_lds_direct"),                        # 9.0 / 9.8
    (40, 64, 14, 14, 384, "tile_lds_direct"),                        # 9.3 / 9.9
    (64, 64, 12, 12, 512, "tile_window"),                            # 14.2 / 12.4
])
def test_dense_runs_take_the_cheaper_kernel(n, cin, h, w, cout, want):
    spec = spec_of(n, cin, h, w, cout)
    layer = R.ConvLayer(spec, np.zeros((cout, 3, 3, cin), np.float32), np.zeros(cout, np.float32), np.ones(spec.m, np.uint8), check_count=False)
    assert B.sparse_conv_plan_kernel(layer.plan, 1) == want


@pytest.mark.parametrize("n,cin,h,w,cout,sp,want", [
    (17, 32, 14, 15, 40, 0.7, "tile_masked_store"),                  # 6.3 us, in this kernel 6.6 and 6.9
    (10, 48, 7, 12, 224, 0.7, "tile_masked_store"),                  # 6.6 / 6.7
    (17, 32, 14, 15, 40, 0.5, "tile_window"),
])
def test_sparse_tiles_are_priced_with_the_rows_between_theirs(n, cin, h, w, cout, sp, want):
    spec = spec_of(n, cin, h, w, cout, sp=sp)
    mask = (np.random.default_rng(5).permutation(spec.m) >= round(sp * spec.m)).astype(np.uint8)
    layer = R.ConvLayer(spec, np.zeros((cout, 3, 3, cin), np.float32), np.zeros(cout, np.float32), mask, check_count=False)
    assert B.sparse_conv_plan_kernel(layer.plan, 0) == want

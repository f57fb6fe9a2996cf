"""The one-launch row tables of a plan (row list, mask copy, band tables, slab spans) at the edges of its segments, against the
compaction of the oracle and, through the kernels that read the band tables, against the layer's oracle."""
import threading

import numpy as np
import pytest
import torch

import workloads as W
from oracle import oracle
from paper_2309_06626_amd import binding as B
from paper_2309_06626_amd import runtime as R
from parity import check_layer, row_mask

pytestmark = pytest.mark.gpu

def masks(rng, length):
    yield np.ones(length, np.uint8)
    yield np.zeros(length, np.uint8)
    yield (rng.random(length) < 0.5).astype(np.uint8)
    m = np.zeros(length, np.uint8)
    m[[0, length - 1]] = 1
    yield m


@pytest.mark.parametrize("n,h,w,mode", [
    (1, 1, 1, "row"), (1, 32, 32, "row"), (1, 25, 41, "row"), (3, 97, 211, "row"),          # below, at and past a segment
    (5, 57, 131, "spatial"), (2, 128, 128, "spatial"), (40, 1, 1023, "spatial"),              # images across segments
    (1, 256, 512, "row"), (1, 257, 512, "row"),                                               # the largest map, and one past it
])
def test_row_list_and_mask_copy(n, h, w, mode):
    spec = W.ConvSpec("t", n=n, c_in=8, h=h, w=w, c_out=8, kh=1, kw=1, pad_h=0, pad_w=0, mask_mode=mode, sparsity=0.0)
    rng = np.random.default_rng(n * h + w)
    ci = W.make_conv_inputs(spec, 3)
    layer = R.ConvLayer(spec, ci.w, ci.bias, ci.mask, check_count=False)
    for m in masks(rng, spec.mask_len):
        for shift in (0, 3):                                       # (a mask need not be aligned)
            dev = torch.from_numpy(np.concatenate([np.zeros(shift, np.uint8), m * 7])).cuda()[shift:]
            B.sparse_conv_plan_set_mask(layer.plan, dev)
            want = oracle.compact_rows(row_mask(spec, m))
            assert B.sparse_conv_plan_info(layer.plan)["kept"] == want.size
            if want.size:
                assert np.array_equal(B.plan_row_idx(layer.plan).cpu().numpy(), want)


@pytest.mark.parametrize("case", [
    dict(n=9, c_in=32, h=57, w=41, c_out=32, kernel="tap"),                     # bands of rows across two segments
    dict(n=7, c_in=64, h=56, w=57, c_out=64, kernel="alternating"),             # bands cut in two
    dict(n=3, c_in=16, h=90, w=83, c_out=16, kernel="single", dtype="f16"),
    dict(n=2, c_in=3, h=150, w=152, c_out=64, k=7, s=2, kernel=None),           # the small-channel band kernel
])
@pytest.mark.parametrize("mode", ["row", "spatial"])
def test_band_tables_across_segments(case, mode, monkeypatch):
    case = dict(case)
    kernel, k, s = case.pop("kernel"), case.pop("k", 3), case.pop("s", 1)
    if kernel:
        monkeypatch.setenv("SPARSE_CONV_BAND_KERNEL", kernel)
    spec = W.ConvSpec("t", kh=k, kw=k, stride_h=s, stride_w=s, pad_h=k // 2, pad_w=k // 2, sparsity=0.4, mask_mode=mode,
                      **{"dtype": "bf16", **case})
    layer = check_layer(W.make_conv_inputs(spec, 17), tiles=(-1, 0) if kernel else None, sample_rows=600)
    assert "band" in B.sparse_conv_plan_kernel(layer.plan, 0)


@pytest.mark.parametrize("n,h,w", [(2, 14, 14), (11, 40, 41)])                  # spans inside the share of one workgroup, and across those of several
def test_slab_spans(n, h, w):
    spec = W.ConvSpec("t", n=n, c_in=64, h=h, w=w, c_out=128, sparsity=0.6)
    layer = check_layer(W.make_conv_inputs(spec, 23), sample_rows=400, options={B.SC_OPT_SLAB: 2})
    assert B.sparse_conv_plan_kernel(layer.plan, 0) == "tile_slab"


@pytest.mark.parametrize("case", [
    dict(n=3, c_in=8, h=97, w=211, c_out=8, kh=1, kw=1, pad_h=0, pad_w=0),           # rows alone
    dict(n=9, c_in=32, h=57, w=41, c_out=32, pad_h=1, pad_w=1),                       # band tables
    dict(n=2, c_in=64, h=14, w=14, c_out=128, slab=True),                             # spans inside one workgroup's share
    dict(n=11, c_in=64, h=40, w=41, c_out=128, slab=True),                            # and across those of several
])
def test_counts_copied_from_the_device_equal_those_in_host_memory(case, monkeypatch):
    """The path of a call that has no slot of host memory: the same plan, the same bits."""
    case = dict(case)
    options = {B.SC_OPT_SLAB: 2} if case.pop("slab", False) else {}
    spec = W.ConvSpec("t", sparsity=0.6, **case)
    ci, other = W.make_conv_inputs(spec, 29), W.make_conv_inputs(spec, 30)
    x, got = R.to_device(ci.x, spec.dtype), []
    for slots in ("1", "0"):
        monkeypatch.setenv("SPARSE_CONV_HOST_SLOTS", slots)
        layer = check_layer(ci, sample_rows=300, options=options)
        B.sparse_conv_plan_set_mask(layer.plan, torch.from_numpy(other.mask).cuda())
        want = oracle.compact_rows(row_mask(spec, other.mask))
        assert np.array_equal(B.plan_row_idx(layer.plan).cpu().numpy(), want)
        got.append((B.sparse_conv_plan_kernel(layer.plan, 0), B.sparse_conv_plan_tiles(layer.plan, 0), R.bits_of(layer.sparse(x)).tobytes()))
    assert got[0] == got[1]


def test_refreshes_of_several_threads_at_once():
    """Plans refreshed by eight threads on streams of their own: every call finds its own counts."""
    def work(i):
        try:
            rng = np.random.default_rng(40 + i)
            spec = W.ConvSpec("t", n=1 + i, c_in=32, h=21 + i, w=30, c_out=32, pad_h=1, pad_w=1, sparsity=0.5)
            ci = W.make_conv_inputs(spec, 41 + i)
            with torch.cuda.stream(torch.cuda.Stream()):
                layer = R.ConvLayer(spec, ci.w, ci.bias, ci.mask, check_count=False)
                for _ in range(40):
                    m = (rng.random(spec.mask_len) < rng.random()).astype(np.uint8)
                    B.sparse_conv_plan_set_mask(layer.plan, torch.from_numpy(m).cuda())
                    want = oracle.compact_rows(row_mask(spec, m))
                    assert B.sparse_conv_plan_info(layer.plan)["kept"] == want.size
                    if want.size:
                        assert np.array_equal(B.plan_row_idx(layer.plan).cpu().numpy(), want)
        except BaseException as e:              # noqa: BLE001 -- reported below, in the test's own thread
            failed.append(e)

    failed = []
    threads = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed[0]

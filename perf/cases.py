"""The workloads whose speed is measured: what a user has this framework do, through its public entry points.

Inference of single layers (16-bit and 32-bit, both tensor layouts, channel counts of trained and of pruned networks, compact
row formats), of a whole network, one training step of a layer in each arithmetic, and the redrawing of a network's masks.

    listed()             the cases
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  inputs, plans and buffers as a user's program holds them before the call
    run(state)           one pass; returns its outputs
    work(case)           bytes and operations that a pass cannot do without
    tolerance(case)      how far two correct implementations may differ
    exact(case, seed)    the outputs in 64 bits, without this package
"""
import math
from dataclasses import dataclass

import numpy as np
import torch

from paper_2309_06626_amd import binding as B
from paper_2309_06626_amd import runtime as R

DEVICE = "cuda:0"
BYTES = {"f32": 4, "f16": 2, "bf16": 2}
TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


# ---- the cases ---------------------------------------------------------------------------------------------------------


def conv(kind="conv", n=1, ci=16, h=16, w=16, co=16, k=3, stride=1, dtype="bf16", layout="nhwc", relu=True, s=0.5,
         mask="row", rows="dense", **more):
    """One layer with a k x k window and "same" padding.  rows = "compact": kept-row matrices in and out (pointwise layers)."""
    return dict(kind=kind, n=n, ci=ci, h=h, w=w, co=co, k=k, stride=stride, dtype=dtype, layout=layout, relu=relu, s=s,
                mask=mask, rows=rows, **more)


def listed():
    return [
        # the smallest call: one image, the paper's own arithmetic; what counts is the latency of a launch
        conv(name="conv3x3_16_f32_n1", n=1, ci=16, h=16, w=16, co=16, dtype="f32"),
        # the layer that `bench.py` measures: first stage of a ResNet18 body at batch 32
        conv(name="conv3x3_64_bf16_n32", n=32, ci=64, h=56, w=56, co=64),
        # last stage of the same body at batch 64: few positions, a long contraction
        conv(name="conv3x3_512_bf16_n64", n=64, ci=512, h=7, w=7, co=512),
        # expansion layer of a MobileNet-style body: little arithmetic, many bytes; the 2-D mask that all images share
        conv(name="conv1x1_96_576_bf16_n64", n=64, ci=96, h=56, w=56, co=576, k=1, mask="spatial"),
        # depthwise layer of the same body
        conv("depthwise", name="depthwise_144_bf16_n64", n=64, ci=144, h=56, w=56, co=144, mask="spatial"),
        # 32-bit inference, the arithmetic the paper measures, on the layer of `bench.py`
        conv(name="conv3x3_64_f32_n32", n=32, ci=64, h=56, w=56, co=64, dtype="f32"),
        # a channel-pruned network run as it is, without rounding its channel counts up
        conv(name="conv3x3_102_f16_n64", n=64, ci=102, h=28, w=28, co=102, dtype="f16", s=0.3),
        # tensors in the channels-first layout, as an exported model holds them
        conv(name="conv3x3_128_nchw_f32_n32", n=32, ci=128, h=28, w=28, co=128, dtype="f32", layout="nchw"),
        # one training step of a layer: new filters into the plans, forward, all three gradients
        conv("train", name="train3x3_128_bf16_n64", n=64, ci=128, h=28, w=28, co=128, mask="spatial"),
        # the same in 32 bits (second convolution of a residual block: no activation of its own)
        conv("train", name="train3x3_64_f32_n16", n=16, ci=64, h=56, w=56, co=64, dtype="f32", relu=False, mask="spatial"),
        # new masks for all resolutions of a network from one score, and the plans told of them
        dict(kind="masks", name="masks_224", res=224, s=0.5),
        # a whole network: the twenty convolutions of a ResNet18 body, pooling and shortcut sums
        dict(kind="network", name="resnet18_bf16_n64", n=64, res=224, dtype="bf16", s=0.5),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cap(c, flops, nbytes):
    """Batch of a drawn layer cut until a pass costs no more than the largest listed one of its kind."""
    while c["n"] > 1:
        w = work(c)
        if w["flops"] <= flops and w["bytes"] <= nbytes:
            break
        c["n"] = max(1, c["n"] * 2 // 3)
    return c


def draw(rng):
    what = rng.choice(["conv", "conv", "pointwise", "depthwise", "f32", "f32", "pruned", "nchw", "train", "train", "masks", "network"])
    s = rng.choice([0.0, 0.25, 0.3, 0.5, 0.5, 0.7])
    mask = rng.choice(["row", "spatial"])
    half = rng.choice(["bf16", "bf16", "f16"])
    if what == "masks":
        return dict(kind="masks", res=32 * _log(rng, 5, 20), s=s or 0.5)
    if what == "network":
        return dict(kind="network", n=_log(rng, 1, 48), res=32 * _log(rng, 4, 7), dtype=half, s=s or 0.5)
    hw = _log(rng, 7, 80)
    h, w = hw, max(5, hw + rng.choice([0, 0, 0, -2, 1, 5]))
    n = _log(rng, 1, 64)
    if what == "depthwise":
        c = 8 * _log(rng, 4, 120)
        return _cap(conv("depthwise", n=n, ci=c, h=h, w=w, co=c, stride=rng.choice([1, 1, 2]), dtype=half, s=s, mask=mask), 6e8, 1.2e8)
    if what == "pointwise":
        return _cap(conv(n=n, ci=16 * _log(rng, 2, 36), h=h, w=w, co=16 * _log(rng, 2, 36), k=1, dtype=half, s=s, mask=mask,
                         relu=rng.random() < 0.5, rows=rng.choice(["dense", "dense", "compact"])), 1.2e10, 2.5e8)
    k, stride = rng.choice([(3, 1), (3, 1), (3, 2), (1, 1)])
    if what == "conv":
        return _cap(conv(n=n, ci=16 * _log(rng, 1, 32), h=h, w=w, co=16 * _log(rng, 1, 32), k=rng.choice([3, 3, 3, 5]),
                         stride=stride, dtype=half, s=s, mask=mask), 1.2e10, 2e8)
    if what == "f32":
        return _cap(conv(n=n, ci=8 * _log(rng, 1, 48), h=h, w=w, co=8 * _log(rng, 1, 48), k=k, stride=stride, dtype="f32", s=s,
                         mask=mask), 4e9, 1e8)
    if what == "pruned":
        return _cap(conv(n=n, ci=_log(rng, 13, 410), h=h, w=w, co=_log(rng, 13, 410), k=k, stride=stride, dtype=rng.choice([half, half, "f32"]),
                         s=s, mask=mask), 4e9, 1e8)
    if what == "nchw":
        return _cap(conv(n=n, ci=_log(rng, 3, 256), h=h, w=w, co=8 * _log(rng, 1, 32), k=k, stride=stride, dtype=rng.choice([half, "f32"]),
                         layout="nchw", s=s, mask=mask), 4e9, 1e8)
    dtype = rng.choice([half, half, "f32"])
    return _cap(conv("train", n=n, ci=8 * _log(rng, 2, 48), h=h, w=w, co=8 * _log(rng, 2, 48), k=k, stride=stride, dtype=dtype,
                     relu=dtype != "f32", s=s, mask=mask), 3e9 if dtype == "f32" else 1.2e10, 1e8)


# ---- layers --------------------------------------------------------------------------------------------------------------


def _out(c):
    p = c["k"] // 2
    return (c["h"] + 2 * p - c["k"]) // c["stride"] + 1, (c["w"] + 2 * p - c["k"]) // c["stride"] + 1


def _keep(s, length):
    return int(math.floor((1.0 - s) * length + 0.5))


def _dw(c):
    return c["kind"] == "depthwise"


def _gen(seed, which):
    return torch.Generator(device=DEVICE).manual_seed(1000003 * int(seed) + which)


def _inputs(c, seed):
    """x = max(N(0,1), 0) as behind an activation, Kaiming-normal filters, a mask with exactly the kept share of ones."""
    t = TORCH[c["dtype"]]
    ho, wo = _out(c)
    n, ci, co, k = c["n"], c["ci"], c["co"], c["k"]
    cg = 1 if _dw(c) else ci
    normal = lambda shape, which: torch.randn(shape, generator=_gen(seed, which), device=DEVICE)
    x = normal((n, ci, c["h"], c["w"]) if c["layout"] == "nchw" else (n, c["h"], c["w"], ci), 0).clamp_(min=0).to(t)
    w = (normal((co, cg, k, k) if c["layout"] == "nchw" else (co, k, k, cg), 1) * math.sqrt(2.0 / (cg * k * k))).to(t)
    bias = normal((co,), 2) * 0.1
    length = ho * wo * (n if c["mask"] == "row" else 1)
    mask = torch.ones(length, dtype=torch.uint8, device=DEVICE)
    mask[torch.randperm(length, generator=_gen(seed, 3), device=DEVICE)[: length - _keep(c["s"], length)]] = 0
    if c["rows"] == "compact":  # the kept rows of x alone
        kept = _kept_rows(c, mask)
        x = x.reshape(-1, ci)[kept].contiguous()
    dy = normal((n, ho, wo, co), 4).to(t) if c["kind"] == "train" else None
    return x, w, bias, mask, dy


def _kept_rows(c, mask):
    return (mask if c["mask"] == "row" else mask.repeat(c["n"])).nonzero().flatten()


def _desc(c):
    return B.make_desc(c["n"], c["ci"], c["h"], c["w"], c["co"], c["k"], c["k"], c["stride"], c["stride"], c["k"] // 2, c["k"] // 2,
                       groups=c["ci"] if _dw(c) else 1, dtype=B.DTYPE_CODE[c["dtype"]],
                       layout=B.SC_NCHW if c["layout"] == "nchw" else B.SC_NHWC, has_bias=1, relu=c["relu"],
                       mask_mode=B.SC_MASK_SPATIAL if c["mask"] == "spatial" else B.SC_MASK_ROW, sparsity=c["s"])


def _exact_conv(c, x, w, bias, mask):
    """The masked convolution in 64 bits, channels last, one window tap at a time; dropped positions hold zeros."""
    ho, wo = _out(c)
    p, st = c["k"] // 2, c["stride"]
    xp = torch.nn.functional.pad(x.double(), (0, 0, p, p, p, p))
    y = bias.double().expand(c["n"], ho, wo, c["co"]).clone()
    for ky in range(c["k"]):
        for kx in range(c["k"]):
            tap = xp[:, ky: ky + st * (ho - 1) + 1: st, kx: kx + st * (wo - 1) + 1: st, :]
            if _dw(c):
                y += tap * w[:, ky, kx, 0].double()
            else:
                y += (tap.reshape(-1, c["ci"]) @ w[:, ky, kx, :].double().t().contiguous()).view_as(y)
    if c["relu"]:
        y.clamp_(min=0)
    m = mask.view(-1 if c["mask"] == "row" else 1, ho, wo, 1).double()
    return y * m, m


# ---- networks ------------------------------------------------------------------------------------------------------------


@dataclass(frozen=True)
class Spec:
    """One convolution of a network, as the package's layer and network drivers read it."""
    name: str
    n: int
    c_in: int
    h: int
    w: int
    c_out: int
    kh: int
    stride_h: int
    relu: bool
    dtype: str
    sparsity: float
    index: int
    layout: str = "nhwc"
    has_bias: bool = True
    mask_mode: str = "row"
    groups: int = 1
    dil_h: int = 1
    dil_w: int = 1

    kw = property(lambda self: self.kh)
    stride_w = property(lambda self: self.stride_h)
    pad_h = property(lambda self: self.kh // 2)
    pad_w = property(lambda self: self.kh // 2)
    ho = property(lambda self: (self.h + 2 * self.pad_h - self.kh) // self.stride_h + 1)
    wo = property(lambda self: (self.w + 2 * self.pad_w - self.kh) // self.stride_w + 1)
    m = property(lambda self: self.n * self.ho * self.wo)

    def y_shape(self):
        return (self.n, self.ho, self.wo, self.c_out)

    def case(self):
        return conv(n=self.n, ci=self.c_in, h=self.h, w=self.w, co=self.c_out, k=self.kh, stride=self.stride_h, dtype=self.dtype,
                    relu=self.relu, s=self.sparsity)


@dataclass(frozen=True)
class Op:
    kind: str
    out: str
    src: str
    src2: str = ""
    spec: Spec = None


def _resnet18(c):
    """The op list of a ResNet18 body: every convolution with its own row mask, batch norm folded into the bias."""
    ops = []

    def add(name, src, ci, co, hw, k, stride, relu):
        ops.append(Op("conv", name, src, spec=Spec(name, c["n"], ci, hw, hw, co, k, stride, relu, c["dtype"], c["s"], len(ops))))
        return ops[-1].spec.ho

    hw = add("stem", "input", 3, 64, c["res"], 7, 2, True)
    ops.append(Op("maxpool", "pool", "stem"))
    hw, src, ci = (hw + 2 - 3) // 2 + 1, "pool", 64
    for stage, co in enumerate((64, 128, 256, 512)):
        for block in range(2):
            stride = 2 if stage and not block else 1
            tag = "l%db%d" % (stage + 1, block)
            out = add(tag + "_conv1", src, ci, co, hw, 3, stride, True)
            add(tag + "_conv2", tag + "_conv1", co, co, out, 3, 1, False)
            short = src
            if stride == 2:
                add(tag + "_down", src, ci, co, hw, 1, 2, False)
                short = tag + "_down"
            ops.append(Op("add_relu", tag, tag + "_conv2", short))
            src, ci, hw = tag, co, out
    return ops


STAGES = ("l1b1", "l2b1", "l3b1", "l4b1")  # results of the four stages


def _network_inputs(c, seed, ops):
    rng = np.random.default_rng(seed)
    x = torch.randn((c["n"], c["res"], c["res"], 3), generator=_gen(seed, 0), device=DEVICE).to(TORCH[c["dtype"]])
    params = {}
    for op in ops:
        if op.kind == "conv":
            sp = op.spec
            w = rng.standard_normal((sp.c_out, sp.kh, sp.kw, sp.c_in), dtype=np.float32) * np.float32(math.sqrt(2.0 / (sp.c_in * sp.kh * sp.kw)))
            mask = np.ones(sp.m, np.uint8)
            mask[rng.permutation(sp.m)[: sp.m - _keep(c["s"], sp.m)]] = 0
            params[sp.name] = (w, rng.standard_normal(sp.c_out, dtype=np.float32) * np.float32(0.1), mask)
    return x, params


# ---- masks ---------------------------------------------------------------------------------------------------------------


def _resolutions(c):
    """Layer resolutions of a body that halves its input five times, with the layer that a plan is kept for."""
    return [(c["res"] >> (i + 1), min(512, 32 << i)) for i in range(5)]


def _score(c, seed):
    return torch.rand((c["res"], c["res"]), generator=_gen(seed, 0), device=DEVICE)


# ---- what is asked of this file -----------------------------------------------------------------------------------------------


def prepare(c, seed):
    if c["kind"] == "network":
        ops = _resnet18(c)
        x, params = _network_inputs(c, seed, ops)
        layers = {name: R.ConvLayer(next(o.spec for o in ops if o.out == name), *p) for name, p in params.items()}
        return dict(kind="network", runner=R.NetworkRunner(ops, {"input": x}, layers), layers=layers)
    if c["kind"] == "masks":
        state = dict(kind="masks", score=_score(c, seed), s=c["s"], layers=[])
        for hw, ch in _resolutions(c):
            lc = conv(n=1, ci=ch, h=hw, w=hw, co=ch, s=c["s"], mask="spatial")
            _, w, _, mask, _ = _inputs(lc, seed + 17)
            workspace = torch.empty(B.sparse_mask_workspace_bytes(hw, hw), dtype=torch.uint8, device=DEVICE)
            state["layers"].append((hw, torch.empty((hw, hw), dtype=torch.uint8, device=DEVICE), workspace, B.sparse_conv_plan(_desc(lc), mask, w)))
        return state
    x, w, bias, mask, dy = _inputs(c, seed)
    ho, wo = _out(c)
    plan = B.sparse_conv_plan(_desc(c), mask, w)
    t = TORCH[c["dtype"]]
    if c["rows"] == "compact":
        y = torch.empty((x.shape[0], c["co"]), dtype=t, device=DEVICE)
        return dict(kind="conv", call=B.prepared_run_rows(plan, x, bias, y, B.SC_ROWS_COMPACT, B.SC_ROWS_COMPACT))
    y = torch.empty((c["n"], c["co"], ho, wo) if c["layout"] == "nchw" else (c["n"], ho, wo, c["co"]), dtype=t, device=DEVICE)
    if c["kind"] != "train":
        return dict(kind="conv", call=B.prepared_run(plan, x, bias, y))
    return dict(kind="train", x=x, w=w, bias=bias, dy=dy, y=y, dx=torch.empty_like(x), plan=plan, back=B.sparse_conv_backward_plan(plan, w),
                dw=torch.empty(w.shape, dtype=torch.float32, device=DEVICE), db=torch.empty(c["co"], dtype=torch.float32, device=DEVICE))


def run(state):
    if state["kind"] == "conv":
        return state["call"]()
    if state["kind"] == "network":
        tensors = state["runner"].run()
        return {name: tensors[name] for name in STAGES}
    if state["kind"] == "masks":
        out = []
        for hw, mask, workspace, plan in state["layers"]:
            B.sparse_mask_generate(state["score"], hw, hw, state["s"], mask, workspace)
            B.sparse_conv_plan_set_mask(plan, mask)
            out.append((mask, B.plan_row_idx(plan)))
        return out
    st = state
    B.sparse_conv_plan_set_filters(st["plan"], st["w"])
    B.sparse_conv_backward_set_filters(st["back"], st["w"])
    B.sparse_conv_run(st["plan"], st["x"], st["bias"], st["y"])
    B.sparse_conv_backward_run(st["back"], st["x"], st["y"], st["dy"], st["dx"], st["dw"], st["db"])
    return {k: st[k] for k in ("y", "dx", "dw", "db")}


def work(c):
    """Every input read once, every output written once; operations of the kept rows."""
    if c["kind"] == "network":
        parts = [work(o.spec.case()) for o in _resnet18(c) if o.kind == "conv"]
        return {"bytes": sum(p["bytes"] for p in parts), "flops": sum(p["flops"] for p in parts)}
    if c["kind"] == "masks":
        return {"bytes": 4 * c["res"] ** 2 + sum((1 + 4 * (1 - c["s"])) * hw * hw for hw, _ in _resolutions(c)), "flops": 5 * c["res"] ** 2}
    ho, wo = _out(c)
    eb, m = BYTES[c["dtype"]], c["n"] * ho * wo
    kept = _keep(c["s"], m) if c["mask"] == "row" else c["n"] * _keep(c["s"], ho * wo)
    k = c["k"] ** 2 * (1 if _dw(c) else c["ci"])
    flops = 2 * kept * k * c["co"]
    length = m if c["mask"] == "row" else ho * wo
    if c["rows"] == "compact":
        return {"bytes": eb * (kept * (c["ci"] + c["co"]) + k * c["co"]) + 4 * c["co"], "flops": flops}
    x, y, w = c["n"] * c["h"] * c["w"] * c["ci"], m * c["co"], k * c["co"]
    if c["kind"] == "train":  # x, w, dy in; y, dx, dw, db out; forward and the two gradients
        return {"bytes": eb * (2 * x + w + 2 * y) + 4 * w + 8 * c["co"] + length, "flops": 3 * flops}
    return {"bytes": eb * (x + y + w) + 4 * c["co"] + length, "flops": flops}


def tolerance(c):
    if c["kind"] == "masks":
        return "exact"
    # about four times the error against 64 bits: 1.7e-3 (bf16), 2.1e-4 (f16), 4e-7 (f32, windows of about a thousand entries);
    # twenty layers one behind the other reach 5.9e-3 (bf16) and 6.7e-4 (f16)
    return {"rel": {"f32": 2e-6, "f16": 8.5e-4, "bf16": 7e-3}[c["dtype"]] * (3.5 if c["kind"] == "network" else 1)}


def exact(c, seed):
    if c["kind"] == "network":
        return _exact_network(c, seed)
    if c["kind"] == "masks":
        return _exact_masks(c, seed)
    x, w, bias, mask, dy = _inputs(c, seed)
    if c["rows"] == "compact":
        y = x.double() @ w.reshape(c["co"], -1).double().t().contiguous() + bias.double()
        return y.clamp_(min=0) if c["relu"] else y
    if c["layout"] == "nchw":
        x, w = x.permute(0, 2, 3, 1), w.permute(0, 2, 3, 1)
    y, m = _exact_conv(c, x, w, bias, mask)
    if c["layout"] == "nchw":
        return y.permute(0, 3, 1, 2).contiguous()
    if c["kind"] != "train":
        return y
    g = dy.double() * m
    if c["relu"]:
        g *= y > 0
    ho, wo = _out(c)
    p, st, ci = c["k"] // 2, c["stride"], c["ci"]
    xp = torch.nn.functional.pad(x.double(), (0, 0, p, p, p, p))
    dxp, dw, g2 = torch.zeros_like(xp), torch.zeros(w.shape, dtype=torch.float64, device=DEVICE), g.reshape(-1, c["co"])
    for ky in range(c["k"]):
        for kx in range(c["k"]):
            at = (slice(None), slice(ky, ky + st * (ho - 1) + 1, st), slice(kx, kx + st * (wo - 1) + 1, st))
            dw[:, ky, kx, :] = g2.t().contiguous() @ xp[at].reshape(-1, ci)
            dxp[at] += (g2 @ w[:, ky, kx, :].double().contiguous()).view(c["n"], ho, wo, ci)
    return {"y": y, "dx": dxp[:, p: p + c["h"], p: p + c["w"], :].contiguous(), "dw": dw, "db": g2.sum(0)}


def _exact_network(c, seed):
    ops = _resnet18(c)
    x, params = _network_inputs(c, seed, ops)
    t = {"input": x.double()}
    for op in ops:
        if op.kind == "conv":
            w, bias, mask = params[op.out]
            w = torch.from_numpy(w).to(TORCH[c["dtype"]]).to(DEVICE)
            t[op.out] = _exact_conv(op.spec.case(), t[op.src], w, torch.from_numpy(bias).to(DEVICE), torch.from_numpy(mask).to(DEVICE))[0]
        elif op.kind == "maxpool":
            a = torch.nn.functional.pad(t[op.src], (0, 0, 1, 1, 1, 1), value=-math.inf)
            ho, wo = (a.shape[1] - 3) // 2 + 1, (a.shape[2] - 3) // 2 + 1
            t[op.out] = torch.stack([a[:, i: i + 2 * ho - 1: 2, j: j + 2 * wo - 1: 2] for i in range(3) for j in range(3)]).amax(0)
        else:
            t[op.out] = (t[op.src] + t[op.src2]).clamp_(min=0)
    return {name: t[name] for name in STAGES}


def _exact_masks(c, seed):
    """Average pooling (its sums: the scores are multiples of 2^-24, so 64 bits hold them exactly) and a stable ranking."""
    score, out = _score(c, seed).double(), []
    for hw, _ in _resolutions(c):
        r = c["res"] // hw
        sums = score[: hw * r, : hw * r].reshape(hw, r, hw, r).sum((1, 3)).flatten()
        mask = torch.ones(hw * hw, dtype=torch.uint8, device=DEVICE)
        mask[torch.argsort(sums, stable=True)[: hw * hw - _keep(c["s"], hw * hw)]] = 0
        out.append((mask.view(hw, hw), mask.nonzero().flatten().to(torch.int32)))
    return out

"""What the privatisation path is asked to do in use, as cases that can be timed.

Two kinds of case:

  "step"   one optimiser step of a layer set through `PrivatiseStep`.  `issue` says how the program drives it: "replay" records
           the step once on persistent input buffers and replays the graph (what bench.py does), "run" hands over the inputs of all
           micro-steps call by call, "micro_steps" hands over one micro-step after the other, as a backward pass produces them.
  "layer"  one layer through the C ABI's own calls (per-example gradients and norms, clipped sum, noise), for programs that own
           their sequencing.  `form` is the form of the clipped sum: "materialise" keeps the per-example gradients,
           "recompute" contracts a second time.

Sizes come from the workloads of this repository (the paper's networks) and from the geometries its tests cover.
"""
from __future__ import annotations

from dataclasses import replace

import torch

import paper_2109_12191_amd as dp
from workloads import get_workload
from workloads.device import make_device_inputs
from workloads.layers import Layer

DEVICE = "cuda:0"


def _step(workload, n, accum, issue, streams=1, hw=0, dtype="", clip="", clip_unit=1, noise="once", momentum=-1.0):
    """A "step" case.  hw 0: the workload's own resolution; dtype and clip "": the workload's own; momentum >= 0: the SGD step
    is fused into finalize."""
    return dict(kind="step", workload=workload, n=n, accum=accum, issue=issue, streams=streams, hw=hw, dtype=dtype, clip=clip,
                clip_unit=clip_unit, noise=noise, momentum=momentum)


def _layer(op, n, cin, cout, h, w, k=1, stride=1, bias=False, groups=0, dtype="f32", form="materialise", nhwc=False):
    """A "layer" case.  dense: h tokens per example, w = 1; conv: k x k, padding (k - 1) / 2; gn: cout == cin, `groups` groups."""
    return dict(kind="layer", op=op, n=n, cin=cin, cout=cout, h=h, w=w, k=k, stride=stride, bias=bias, groups=groups,
                dtype=dtype, form=form, nhwc=nhwc)


def listed():
    return [
        # the smallest step: a two-layer fp32 classifier, every call issued from the host
        dict(name="mlp_f32_run", **_step("mlp", 32, 1, "run")),
        # one fp32 convolution with bias, accumulated over four micro-batches with a bound of its own
        dict(name="conv3x3_f32_run", **_step("conv3x3", 16, 4, "run")),
        # CIFAR-sized fp32 network with GroupNorm gradients: many narrow layers, many examples
        dict(name="resnet20_f32_replay", **_step("resnet20", 256, 1, "replay", streams=8)),
        # CIFAR-sized wide bf16 network with GroupNorm: small maps, many parameters
        dict(name="resnet18_gn_replay", **_step("resnet18_gn", 32, 8, "replay", streams=8)),
        # the benchmark's own step: ImageNet-sized network, micro-batches of 32
        dict(name="resnet50_replay", **_step("resnet50", 32, 8, "replay", streams=8)),
        # the regime the paper is named for: micro-batches of one example, a bound per layer, recorded once and replayed
        dict(name="resnet50_nano_replay", **_step("resnet50_nano", 1, 64, "replay", streams=4)),
        # the same regime as a backward pass drives it, one micro-step after the other, nothing recorded
        dict(name="resnet50_nano_micro_steps", **_step("resnet50_nano", 1, 16, "micro_steps")),
        # a resolution and a micro-batch that nothing was laid out for, GroupNorm gradients, momentum SGD, issued from the host
        dict(name="resnet50_gn_hw200_run", **_step("resnet50_gn", 12, 3, "run", streams=8, hw=200, clip="per_layer", momentum=0.9)),
        # clipping units of four examples (the micro-batch clipping of the paper's GPU baseline)
        dict(name="resnet50_units4_replay", **_step("resnet50", 32, 4, "replay", streams=8, clip_unit=4)),
        # one strided fp32 convolution with bias on a ragged map, called layer by layer
        dict(name="layer_conv5x5_f32", **_layer("conv", 40, 40, 72, 45, 37, k=5, stride=2, bias=True)),
        # a dense layer over several tokens per example, clipped sum recomputed
        dict(name="layer_dense_tokens", **_layer("dense", 16, 768, 768, 128, 1, bias=True, dtype="bf16", form="recompute")),
    ]


# ---- drawn cases: the ranges behind the list ----------------------------------------------------------------------

def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _draw_step(rng):
    name = rng.choice(("mlp", "conv3x3", "resnet20", "resnet18_gn", "resnet50", "resnet50", "resnet50_nano", "resnet50_nano",
                       "resnet50_gn"))
    issue = rng.choice(("replay", "run", "micro_steps"))
    streams = rng.choice((1, 8))
    momentum = rng.choice((-1.0, -1.0, 0.0, 0.9))
    if name == "mlp":
        return _step(name, _log_int(rng, 8, 512), rng.choice((1, 1, 2, 4)), issue, 1, momentum=momentum)
    if name == "conv3x3":
        return _step(name, _log_int(rng, 4, 64), rng.choice((1, 2, 4)), issue, 1, hw=rng.choice((28, 33, 56, 64)),
                     dtype=rng.choice(("f32", "f32", "bf16")), momentum=momentum)
    if name == "resnet20":
        return _step(name, _log_int(rng, 32, 256), rng.choice((1, 2)), issue, streams, momentum=momentum)
    if name == "resnet18_gn":
        unit = rng.choice((1, 1, 1, 2))
        return _step(name, unit * _log_int(rng, 6, 32), rng.choice((1, 2, 4)), issue, streams, hw=rng.choice((32, 32, 24, 40)),
                     dtype=rng.choice(("bf16", "bf16", "bf16", "f32")), clip=rng.choice(("global", "per_layer")), clip_unit=unit,
                     noise=rng.choice(("once", "once", "per_example")) if unit == 1 else "once", momentum=momentum)
    if name == "resnet50_nano":
        n = rng.choice((1, 1, 1, 2))
        return _step(name, n, _log_int(rng, 4, 64) // n, issue, rng.choice((1, 4)), hw=rng.choice((224, 224, 224, 192, 160)),
                     momentum=momentum)
    if name == "resnet50_gn":
        return _step(name, _log_int(rng, 8, 24), rng.choice((1, 2, 3)), issue, streams, hw=rng.choice((224, 200, 176, 160, 128)),
                     clip=rng.choice(("global", "per_layer")), momentum=momentum)
    unit = rng.choice((1, 1, 1, 4))
    return _step(name, 4 * _log_int(rng, 2, 12), rng.choice((1, 2, 4)), issue, streams, hw=rng.choice((224, 224, 224, 192, 208)),
                 clip=rng.choice(("global", "per_layer")), clip_unit=unit, momentum=momentum)


def _draw_layer(rng):
    op = rng.choice(("conv", "conv", "dense"))
    dtype = rng.choice(("f32", "bf16"))
    form = rng.choice(("materialise", "recompute"))
    bias = rng.choice((False, True))
    n = _log_int(rng, 8, 64)
    if op == "dense":
        return _layer(op, n, _log_int(rng, 100, 1024), _log_int(rng, 36, 1024), _log_int(rng, 3, 128), 1, bias=bias, dtype=dtype,
                      form=form)
    return _layer(op, n, _log_int(rng, 8, 160), _log_int(rng, 8, 160), rng.randint(10, 56), rng.randint(10, 56),
                  k=rng.choice((1, 3, 3, 5)), stride=rng.choice((1, 1, 2)), bias=bias, dtype=dtype, form=form,
                  nhwc=rng.random() < 0.25)


def draw(rng):
    return _draw_step(rng) if rng.random() < 0.75 else _draw_layer(rng)


# ---- running them -------------------------------------------------------------------------------------------------

def _workload(case, seed=0):
    wl = get_workload(case["workload"], n=case["n"], accum=case["accum"], hw=case["hw"] or None)
    return replace(wl, dtype=case["dtype"] or wl.dtype, clip_mode=case["clip"] or wl.clip_mode, data_seed=seed)


def _the_layer(case):
    if case["op"] == "conv":
        return Layer("conv", case["cin"], case["cout"], case["h"], case["w"], case["k"], case["k"], case["stride"],
                     (case["k"] - 1) // 2, case["bias"])
    return Layer("dense", case["cin"], case["cout"], case["h"], 1, has_bias=case["bias"])


CLIP_C, SIGMA = 1.0, 1.1          # bound and noise multiplier of the "layer" cases


def prepare(case, seed):
    if case["kind"] == "step":
        wl = _workload(case, seed)
        inputs = make_device_inputs(wl, wl.accum, torch.device(DEVICE))
        ps = dp.PrivatiseStep(wl, device=DEVICE, streams=case["streams"], noise=case["noise"], clip_unit=case["clip_unit"])
        if case["momentum"] >= 0.0:
            ps.enable_update(lr=0.1, momentum=case["momentum"])
        if case["issue"] == "replay":
            ps.capture(inputs)
        return dict(kind="step", issue=case["issue"], ps=ps, inputs=inputs)
    layer = _the_layer(case)
    desc = dp.make_desc(layer, case["n"], case["dtype"], dp.DP_NHWC if case["nhwc"] else dp.DP_NCHW)
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def tensor(shape, std):
        t = torch.randn((case["n"],) + tuple(shape), generator=gen, device=DEVICE) * std
        if case["nhwc"]:
            t = t.permute(0, 2, 3, 1)
        return t.to(dtype).contiguous()

    x, dy = tensor(layer.x_shape, 1.0), tensor(layer.dy_shape, 0.01)
    pw, pb = dp.dp_weight_count(desc), dp.dp_bias_count(desc)
    row = (pw + 3) // 4 * 4 + (pb + 3) // 4 * 4          # weights then bias, each padded to 16 bytes
    materialise = case["form"] == "materialise"
    need = max(16, dp.dp_workspace_bytes(desc, dp.DP_WS_PER_EXAMPLE_GRAD), dp.dp_workspace_bytes(desc, dp.DP_WS_RECOMPUTE))
    f32 = dict(dtype=torch.float32, device=DEVICE)
    return dict(kind="layer", desc=desc, n=case["n"], x=x, dy=dy, pw=pw, pb=pb, row=row, form=case["form"],
                g=torch.zeros((case["n"], row), **f32) if materialise else None,
                sqnorm=torch.zeros(case["n"], **f32), ws=torch.empty(need, dtype=torch.uint8, device=DEVICE),
                acc=torch.zeros(row, **f32), out=torch.zeros(row, **f32),
                tensors=dp.TensorTable([0, row - (pb + 3) // 4 * 4] if pb else [0], [pw, pb] if pb else [pw], [0, 1] if pb else [0]))


def run(state):
    if state["kind"] == "step":
        ps = state["ps"]
        if state["issue"] == "replay":
            ps.replay()
        elif state["issue"] == "run":
            ps.run(state["inputs"])
        else:
            ps.begin_step()
            for inputs in state["inputs"]:
                ps.micro_step(inputs)
            ps.finalize()
        return [ps.out, ps.acc, ps.group_sqnorm, ps.theta, ps.velocity]
    s = state
    desc, n, row, sqnorm, acc = s["desc"], s["n"], s["row"], s["sqnorm"], s["acc"]
    bias_at = s["row"] - (s["pb"] + 3) // 4 * 4
    acc.zero_()
    if s["form"] == "materialise":
        g = s["g"]
        dp.dp_per_example_grad(desc, s["x"], s["dy"], g, g[:, bias_at:] if s["pb"] else None, sqnorm, s["ws"], g_stride=row)
        dp.dp_clip_accumulate(g, sqnorm, CLIP_C, n, row, acc)
    else:
        dp.dp_per_example_grad(desc, s["x"], s["dy"], None, None, sqnorm, s["ws"])
        dp.dp_clip_accumulate_recompute(desc, s["x"], s["dy"], sqnorm, CLIP_C, acc, acc[bias_at:] if s["pb"] else None, s["ws"])
    dp.dp_add_noise_finalize_flat(acc, s["out"], s["tensors"], SIGMA, CLIP_C, n, seed=0)
    return [s["out"], acc, sqnorm, s["g"]]


def work(case):
    """Inputs read once; clipped sum and privatised gradient (and what the fused SGD step updates, and the per-example gradients
    where the caller asks for them) written once.  Operations: one contraction per layer and example."""
    if case["kind"] == "step":
        wl = _workload(case)
        per_param = 8 + (0 if case["momentum"] < 0.0 else 8 if case["momentum"] == 0.0 else 16)
        return {"bytes": wl.in_bytes_per_example * wl.total_batch + per_param * wl.n_params,
                "flops": wl.flops_per_example * wl.total_batch}
    layer = _the_layer(case)
    p = layer.pw + layer.pb
    stored = 4 * case["n"] * p if case["form"] == "materialise" else 0
    return {"bytes": layer.in_bytes(2 if case["dtype"] == "bf16" else 4) * case["n"] + stored + 8 * p,
            "flops": layer.flops * case["n"]}


def tolerance(case):
    dtype = case["dtype"] or get_workload(case["workload"]).dtype
    # Measured between the two forms of the clipped sum, which contract in another order (2-norm, largest over rms): fp32 1.1e-6 and
    # 1.2e-5 over sums of up to 12,544 terms, and the normal deviates are good to about 1e-6; bf16 1.6e-3 and 0.048, because the
    # recomputing form rounds the scaled output gradient to bf16 once more (2^-9 per element) where the other keeps it in fp32.
    return {"rel": 1e-5, "max": 1e-4} if dtype == "f32" else {"rel": 6e-3, "max": 0.2}

"""GPU parity of the whole path (all five steps through the C ABI) against the fp64 oracle,
on the five workloads -- full size where the oracle finishes in seconds, otherwise the same
layer structure on smaller feature maps / fewer examples."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2109_12191_amd as dp
from gpu_util import BF16_TOL, F32_TOL, assert_close, dev, host
from workloads import Workload, conv, get_workload, make_inputs, to_bf16_grid

pytestmark = pytest.mark.gpu


def _run_both(wl, mode):
    steps = [make_inputs(wl, m) for m in range(wl.accum)]
    ref = oracle.privatise(wl, steps)
    ps = dp.PrivatiseStep(wl, mode=mode)
    ps.begin_step()
    n2_gpu = []
    for inputs in steps:
        ps.micro_step([(dev(x, wl.dtype), dev(dy, wl.dtype)) for x, dy in inputs])
        n2_gpu.append(host(ps.group_sqnorm).T.copy())          # [n, G]
    acc_gpu = ps.acc.clone()
    ps.finalize()
    torch.cuda.synchronize()
    return ref, ps, n2_gpu, acc_gpu


def _check(wl, mode):
    tol = F32_TOL if wl.dtype == "f32" else BF16_TOL
    ref, ps, n2_gpu, acc_gpu = _run_both(wl, mode)
    # H2: squared norms per example and group
    for m in range(wl.accum):
        assert np.allclose(n2_gpu[m], ref["n2"][m], rtol=tol, atol=0), f"n2 micro-step {m}"
    # H4: clipped sum before noise, tensor by tensor
    for li, l in enumerate(wl.layers):
        a = host(acc_gpu[ps.off_w[li]: ps.off_w[li] + ps.pw[li]])
        assert_close(a, ref["acc_w"][li], tol, f"acc_w[{li}] {l.name} ({ps.form[li]})")
        if l.pb:
            b = host(acc_gpu[ps.off_b[li]: ps.off_b[li] + ps.pb[li]])
            assert_close(b, ref["acc_b"][li], tol, f"acc_b[{li}] {l.name}")
    # H5: final output
    for li, l in enumerate(wl.layers):
        assert_close(host(ps.out_w(li)), ref["out_w"][li], tol, f"out_w[{li}] {l.name}")
        if l.pb:
            assert_close(host(ps.out_b(li)), ref["out_b"][li], tol, f"out_b[{li}] {l.name}")
    return ps


@pytest.mark.parametrize("mode", ["auto", "materialise", "recompute"])
def test_mlp_workload_full_size(mode):
    _check(get_workload("mlp"), mode)


@pytest.mark.parametrize("mode", ["auto", "recompute"])
def test_conv3x3_workload_full_size(mode):
    _check(get_workload("conv3x3"), mode)


@pytest.mark.parametrize("mode", ["auto", "recompute"])
def test_resnet20_workload(mode):
    # config 3 at full size: 39 layers, 256 examples
    _check(get_workload("resnet20"), mode)


@pytest.mark.parametrize("mode", ["auto", "materialise", "recompute"])
def test_resnet50_layer_set_small_maps(mode):
    # all 54 layers with their real channel counts, 64x64 input instead of 224x224
    ps = _check(get_workload("resnet50", n=4, accum=2, hw=64), mode)
    if mode == "auto":
        assert "materialise" in ps.form or "recompute" in ps.form


def test_resnet50_nano_per_layer_clipping_small_maps():
    wl = get_workload("resnet50_nano", accum=4, hw=64)
    assert wl.n == 1 and wl.n_groups == 54
    _check(wl, "auto")


def test_split_and_resume_gives_same_bits():
    """State between micro-steps is only the accumulator: copy it out and in mid-step."""
    wl = get_workload("conv3x3", n=4, accum=3, hw=14)
    steps = [[(dev(x), dev(dy)) for x, dy in make_inputs(wl, m)] for m in range(3)]
    a = dp.PrivatiseStep(wl)
    a.run(steps)
    b = dp.PrivatiseStep(wl)
    b.begin_step()
    b.micro_step(steps[0])
    saved = b.acc.clone()
    c = dp.PrivatiseStep(wl)
    c.begin_step()
    c.acc.copy_(saved)
    c.micro_step(steps[1])
    c.micro_step(steps[2])
    c.finalize()
    torch.cuda.synchronize()
    assert torch.equal(a.out, c.out)


def test_graph_replay_with_side_streams_matches_eager_every_time():
    """The whole step recorded into a HIP graph (layers spread over side streams) gives the same bits as the
    call-by-call path at the same optimiser step, on every replay, with eager work in between; consecutive
    steps draw different noise (the step counter is a device word that the graph itself advances)."""
    wl = get_workload("resnet50", n=4, accum=2, hw=64)
    steps = [[(dev(x, wl.dtype), dev(dy, wl.dtype)) for x, dy in make_inputs(wl, m)] for m in range(wl.accum)]
    eager = dp.PrivatiseStep(wl, streams=1)
    want = []
    for k in range(3):
        assert eager.step == k
        want.append(eager.run(steps).clone())
    torch.cuda.synchronize()
    assert not torch.equal(want[0], want[1]) and not torch.equal(want[1], want[2])
    g = dp.PrivatiseStep(wl, streams=4)
    g.capture(steps)
    assert g.step == 0
    for rep in range(3):
        g.out.zero_()
        g.acc.fill_(123.0)                 # the graph must clear the accumulator itself
        torch.cuda.synchronize()
        got = g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want[rep]), f"replay {rep}"
        eager.set_step(rep)                # eager work between replays
        again = eager.run(steps)
        torch.cuda.synchronize()
        assert torch.equal(again, want[rep])
    assert g.step == 3 and int(g._step_dev.item()) == 3
    # multi-stream without a graph as well
    ms = dp.PrivatiseStep(wl, streams=3)
    assert torch.equal(ms.run(steps), want[0])


def test_consecutive_optimiser_steps_draw_fresh_noise_and_match_the_oracle():
    """Two optimiser steps in a row on the same data: the released gradients carry different noise, and each
    matches the oracle evaluated at its own step number (eager and graph replay)."""
    from dataclasses import replace
    wl = get_workload("conv3x3", n=4, accum=2, hw=14)
    host_steps = [make_inputs(wl, m) for m in range(wl.accum)]
    refs = [oracle.privatise(replace(wl, step=wl.step + k), host_steps) for k in range(2)]
    steps = [[(dev(x), dev(dy)) for x, dy in inputs] for inputs in host_steps]
    for use_graph in (False, True):
        ps = dp.PrivatiseStep(wl, streams=2 if use_graph else 1)
        if use_graph:
            ps.capture(steps)
        outs = []
        for k in range(2):
            out = ps.replay() if use_graph else ps.run(steps)
            torch.cuda.synchronize()
            outs.append(out.clone())
            for li, l in enumerate(wl.layers):
                assert_close(host(ps.out_w(li)), refs[k]["out_w"][li], F32_TOL, f"graph={use_graph} step {k} out_w")
                assert_close(host(ps.out_b(li)), refs[k]["out_b"][li], F32_TOL, f"graph={use_graph} step {k} out_b")
        diff = host(outs[1] - outs[0])[: ps.pw[0]]
        # the clipped sums cancel; what is left is the difference of two independent noise draws
        sigma_c_over_b = wl.sigma * wl.clip_c / wl.total_batch
        assert abs(diff.std() / (math.sqrt(2.0) * sigma_c_over_b) - 1.0) < 0.05


def test_fused_optimiser_update_over_two_steps():
    """finalize with the SGD step fused in: theta after two optimiser steps (momentum carried) against the
    oracle's finalize + update."""
    wl = get_workload("conv3x3", n=4, accum=2, hw=14)
    steps = [[(dev(x), dev(dy)) for x, dy in make_inputs(wl, m)] for m in range(wl.accum)]
    ref = oracle.privatise(wl, [make_inputs(wl, m) for m in range(wl.accum)])
    ps = dp.PrivatiseStep(wl, streams=2)
    rng = np.random.default_rng(23)
    theta0 = rng.standard_normal(ps.p_total).astype(np.float32)
    ps.enable_update(lr=0.05, momentum=0.9, theta=dev(theta0))
    from dataclasses import replace
    ref1 = oracle.privatise(replace(wl, step=wl.step + 1), [make_inputs(wl, m) for m in range(wl.accum)])
    ps.run(steps)
    ps.set_lr(0.025)
    ps.run(steps)                                    # same data, next optimiser step: fresh noise
    torch.cuda.synchronize()
    for li, l in enumerate(wl.layers):
        for off, cnt, g, g1 in ((ps.off_w[li], ps.pw[li], ref["out_w"][li], ref1["out_w"][li]),
                                (ps.off_b[li], ps.pb[li], ref["out_b"][li], ref1["out_b"][li])):
            if not cnt:
                continue
            th, v = theta0[off: off + cnt].astype(np.float64), np.zeros(cnt)
            th, v = oracle.sgd_update(g.reshape(-1), th, v, 0.05, 0.9)
            th, v = oracle.sgd_update(g1.reshape(-1), th, v, 0.025, 0.9)
            assert_close(host(ps.theta[off: off + cnt]), th, F32_TOL, f"theta layer {li}")
            assert_close(host(ps.out[off: off + cnt]), g1.reshape(-1), F32_TOL, f"gradient layer {li}")


@pytest.mark.parametrize("streams", [1, 3])
def test_per_example_noise_form_whole_path(streams):
    """The paper's as-built form: noise per clipped example, nothing added in finalize."""
    wl = get_workload("resnet50", n=4, accum=2, hw=64)
    host_steps = [make_inputs(wl, m) for m in range(wl.accum)]
    ref = oracle.privatise(wl, host_steps, noise_form="per_example")
    steps = [[(dev(x, wl.dtype), dev(dy, wl.dtype)) for x, dy in inputs] for inputs in host_steps]
    ps = dp.PrivatiseStep(wl, streams=streams, noise="per_example")
    ps.run(steps)
    torch.cuda.synchronize()
    for li, l in enumerate(wl.layers):
        assert_close(host(ps.out_w(li)), ref["out_w"][li], BF16_TOL, f"out_w[{li}] {l.name}")
        if l.pb:
            assert_close(host(ps.out_b(li)), ref["out_b"][li], BF16_TOL, f"out_b[{li}]")


@pytest.mark.parametrize("name,n,accum,hw", [("resnet18_gn", 3, 2, 16), ("resnet50_gn", 2, 1, 64), ("resnet101_gn", 2, 1, 32)])
def test_further_layer_sets_with_groupnorm(name, n, accum, hw):
    """The paper's other networks (ResNet-18-GN, ResNet-101-GN32) and ResNet-50 with its GroupNorm gradients:
    same kernels, more shapes; whole path against the oracle on small maps."""
    wl = get_workload(name, n=n, accum=accum, hw=hw)
    assert any(l.kind == "gn" for l in wl.layers)
    _check(wl, "auto")


def test_both_clip_branches_zero_example_and_infinite_bound():
    """The five workloads clip every example; here the bound is the median norm (half the examples keep their
    gradient), one example is all zeros (factor 1, contributes nothing), and a second run has C = inf, sigma = 0
    (the result is the plain mean gradient)."""
    import math
    from dataclasses import replace
    base = get_workload("resnet50", n=6, accum=2, hw=64)
    host_steps = [make_inputs(base, m) for m in range(base.accum)]
    for li in range(len(base.layers)):                     # example 3 of micro-step 0: all-zero gradient
        host_steps[0][li][1][3] = 0.0
    probe = oracle.privatise(base, host_steps)
    med = float(np.sqrt(np.median(np.concatenate([n2[:, 0] for n2 in probe["n2"]]))))
    for wl in (replace(base, clip_c=med), replace(base, clip_c=math.inf, sigma=0.0)):
        ref = oracle.privatise(wl, host_steps)
        f_all = np.concatenate([f[:, 0] for f in ref["f"]])
        if math.isfinite(wl.clip_c):
            assert (f_all < 1).sum() >= 4 and (f_all == 1).sum() >= 4          # both branches are taken
        steps = [[(dev(x, wl.dtype), dev(dy, wl.dtype)) for x, dy in inputs] for inputs in host_steps]
        for mode in ("auto", "recompute"):
            ps = dp.PrivatiseStep(wl, mode=mode, streams=2)
            ps.begin_step()
            ps.micro_step(steps[0])
            torch.cuda.synchronize()
            assert host(ps.group_sqnorm)[0, 3] == 0.0                           # the zero example
            ps.micro_step(steps[1])
            ps.finalize()
            torch.cuda.synchronize()
            for li, l in enumerate(wl.layers):
                assert_close(host(ps.out_w(li)), ref["out_w"][li], BF16_TOL, f"{mode} C={wl.clip_c} out_w[{li}] {l.name}")


# Sums of the same products in another order: F32_TOL covers the fp32 sums; the squared norms differ in their last bits too (about 1e-6),
# which turns the rounding of the scaled bf16 operands of recomputing layers for one element in 2^9 * 1e-6 (relative error of a sum: at most
# 2^-9 sqrt(5e-4) = 4e-5).
@pytest.mark.parametrize("streams", [1, 3])
@pytest.mark.parametrize("name,n,accum,together", [("resnet18_gn", 3, 3, 3), ("resnet18_gn", 1, 5, 5), ("resnet18_gn", 5, 1, 1), ("resnet18_gn", 3, 0, 1),
                                                   ("resnet18_gn", 3, 5, 2), ("resnet50", 4, 5, 3), ("resnet50_nano", 1, 7, 3), ("resnet20", 5, 3, 2)])
def test_odd_phases_and_empty_steps_match_single_micro_steps(monkeypatch, name, n, accum, together, streams):
    """run() puts the micro-steps of a step together (an odd number of examples, phases of different size, a last phase of one); one after
    the other they give the same sums, the same norms and the same noise."""
    wl = get_workload(name, n=n, accum=max(1, accum), hw=32 if name == "resnet20" else 16 if name == "resnet18_gn" else 64)
    inputs = [[(dev(x, wl.dtype), dev(dy, wl.dtype)) for x, dy in make_inputs(wl, m)] for m in range(accum)]
    want = dp.PrivatiseStep(wl)
    monkeypatch.setattr(dp.PrivatiseStep, "_micro_steps_together", lambda self: together)
    got = dp.PrivatiseStep(wl, streams=streams)
    if accum:
        assert got._phase_sizes(accum)[0] == together
    want.begin_step()
    for step in inputs:
        want.micro_step(step)
    want.finalize()
    for _ in range(2):
        got.set_step(0)
        got.run(inputs)
        torch.cuda.synchronize()
        assert_close(host(got.acc), host(want.acc), F32_TOL, "acc")
        assert_close(host(got.out), host(want.out), F32_TOL, "out")
        if accum:
            assert np.allclose(host(got.group_sqnorm), host(want.group_sqnorm), rtol=F32_TOL)


@pytest.mark.parametrize("name,n,hw,sizes", [("resnet18_gn", 24, 40, [6, 5]), ("resnet50", 4, 64, [3, 3, 2])])
def test_phases_of_different_size_on_side_streams(monkeypatch, name, n, hw, sizes):
    """Plans of different size spread the layers over the streams differently; the sums are those of one stream, bit for bit."""
    wl = get_workload(name, n=n, accum=sum(sizes), hw=hw)
    inputs = [[(dev(x, wl.dtype), dev(dy, wl.dtype)) for x, dy in make_inputs(wl, m)] for m in range(2)]
    steps = [inputs[m % 2] for m in range(wl.accum)]
    monkeypatch.setattr(dp.PrivatiseStep, "_micro_steps_together", lambda self: sizes[0])
    ps = [dp.PrivatiseStep(wl, streams=s) for s in (1, 8, 8)]
    assert all(p._phase_sizes(wl.accum) == sizes for p in ps)
    want = ps[0].run(steps).clone()
    acc = ps[0].acc.clone()
    for _ in range(3):
        ps[1].set_step(0)
        ps[1].run(steps)
        assert torch.equal(ps[1].acc, acc) and torch.equal(ps[1].out, want)
    ps[2].capture(steps)
    for _ in range(3):
        ps[2].set_step(0)
        ps[2].replay()
        assert torch.equal(ps[2].acc, acc) and torch.equal(ps[2].out, want)


def test_two_recorded_steps_and_one_that_the_caller_records():
    """Graphs over different inputs, each replayed after the others were recorded and longer steps were run."""
    wl = get_workload("resnet18_gn", n=2, accum=3, hw=16)
    sets = [[[(dev(x, wl.dtype), dev(dy, wl.dtype)) for x, dy in make_inputs(wl, 3 * k + m)] for m in range(3)] for k in range(3)]
    eager = dp.PrivatiseStep(wl)
    want = []
    for steps in sets:
        eager.set_step(0)
        want.append(eager.run(steps).clone())
    ps = dp.PrivatiseStep(wl, streams=3)
    graphs = [ps.capture(steps) for steps in sets[:2]]
    ps.run(sets[2])
    torch.cuda.synchronize()
    graphs.append(torch.cuda.CUDAGraph())
    with torch.cuda.graph(graphs[2]):
        ps.run(sets[2])
    for _ in range(3):
        ps.run(sets[0] + sets[1])                  # a longer step: a larger table
        for graph, out in zip(graphs, want):
            fill = [torch.full((1 << k,), -1, dtype=torch.int64, device="cuda:0") for k in range(6, 16)]     # whatever was given back
            ps.set_step(0)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(ps.out, out) and all(bool((f == -1).all()) for f in fill)


@pytest.mark.parametrize("name,n,accum,streams", [("resnet50_nano", 1, 5, 1), ("resnet50_nano", 1, 5, 3), ("conv3x3", 4, 3, 2)])
def test_norms_of_the_last_micro_step(name, n, accum, streams):
    """group_sqnorm after a step whose micro-steps were issued together: a contiguous matrix, the last micro-step's numbers, eager and
    replayed."""
    wl = get_workload(name, n=n, accum=accum, hw=32)
    steps = [[(dev(x, wl.dtype), dev(dy, wl.dtype)) for x, dy in make_inputs(wl, m)] for m in range(accum)]
    single, ps = dp.PrivatiseStep(wl), dp.PrivatiseStep(wl, streams=streams)
    assert ps.micro_steps_per_phase == accum
    single.begin_step()
    for inputs in steps:
        single.micro_step(inputs)
    want = single.group_sqnorm.clone()
    ps.run(steps)
    assert ps.group_sqnorm.is_contiguous() and ps.group_sqnorm.shape == want.shape
    assert torch.allclose(ps.group_sqnorm, want, rtol=1e-5, atol=0.0)
    ps.capture(steps)
    for _ in range(3):
        ps.group_sqnorm.zero_()
        ps.replay()
        assert torch.allclose(ps.group_sqnorm, want, rtol=1e-5, atol=0.0)


# Squared norms of finished fp32 gradients: 49 exact products per element, whose partial sums are up to 1 / 1 % of the result here, each rounded by
# 2^-24; errors of elements are as good as independent, and 10^5 of them are squared and added: below 49 * 100 * 2^-24 / sqrt(10^5) = 1e-6, taken
# ten times.  (By way of Gram matrices: 1e-4 and more.)
def _centred(layer, n, seed):
    """X nearly constant over the positions, dY of sum zero over them, on the bf16 grid."""
    rng = np.random.default_rng(seed)
    x = to_bf16_grid(1.0 + 0.01 * rng.standard_normal((n,) + tuple(layer.x_shape)).astype(np.float32))
    dy = rng.integers(-3, 4, (n,) + tuple(layer.dy_shape)).astype(np.float32)
    dy.reshape(n, layer.cout, -1)[:, :, -1] = -dy.reshape(n, layer.cout, -1)[:, :, :-1].sum(-1)
    return x, (dy * 2.0 ** -7).astype(np.float32)


@pytest.mark.parametrize("n,accum,streams", [(1, 12, 1), (2, 6, 3)])
def test_norms_do_not_depend_on_how_many_micro_steps_share_a_phase(n, accum, streams):
    layers = (conv(512, 2048, 1, 1, 7), conv(1024, 1024, 1, 2, 13), conv(512, 256, 3, 1, 7))
    wl = Workload("centred", layers, n, accum, "bf16", "per_layer", 1.0, 1.0, tuple("normal" for _ in layers), 0.01, 7)
    ins = [_centred(l, n * accum, 40 + k) for k, l in enumerate(layers)]
    want = np.stack([[oracle.sqnorm(oracle.example_grad(l, x[i], dy[i])[0]) for i in range(n * accum)] for l, (x, dy) in zip(layers, ins)])
    steps = [[(dev(x[m * n:(m + 1) * n], "bf16"), dev(dy[m * n:(m + 1) * n], "bf16")) for x, dy in ins] for m in range(accum)]
    ps = dp.PrivatiseStep(wl, streams=streams)
    assert ps.micro_steps_per_phase == accum and ps._main.form != ps.form
    ps.run(steps)
    together = host(ps._main.group_sqnorm[0])
    ps.begin_step()
    for m, inputs in enumerate(steps):
        ps.micro_step(inputs)
        for got in (together[:, m * n:(m + 1) * n], host(ps.group_sqnorm)):
            assert np.allclose(got, want[:, m * n:(m + 1) * n], rtol=1e-5, atol=0), (m, got / want[:, m * n:(m + 1) * n] - 1)


@pytest.mark.parametrize("n,accum,streams,layers", [(1, 8, 1, None), (1, 8, 4, None), (2, 5, 4, None),
                                                    (1, 12, 3, (conv(512, 2048, 1, 1, 7), conv(1024, 1024, 1, 2, 13), conv(512, 256, 3, 1, 7)))])
def test_stored_gradients_of_the_last_micro_step(n, accum, streams, layers):
    """g after a step whose micro-steps were issued together, some layers (or all) recomputed: every column, as the micro-step by itself stores it,
    eager and replayed, before and after the next step begins."""
    wl = get_workload("resnet50_nano", n=n, accum=accum, hw=64)
    if layers:
        wl = Workload("all recomputed", layers, n, accum, "bf16", "per_layer", 1.0, 1.0, tuple("normal" for _ in layers), 0.01, 7)
    steps = [[(dev(x, wl.dtype), dev(dy, wl.dtype)) for x, dy in make_inputs(wl, m)] for m in range(accum)]
    single, ps = dp.PrivatiseStep(wl), dp.PrivatiseStep(wl, streams=streams)
    assert ps.micro_steps_per_phase == accum and ps._main.form != ps.form and ("materialise" in ps._main.form) == (layers is None)
    single.begin_step()
    for inputs in steps:
        single.micro_step(inputs)
    want = single.g.clone()
    ps.run(steps)
    for _ in range(2):
        assert ps.g.shape == want.shape and ps.g.is_contiguous()
        assert_close(host(ps.g), host(want), F32_TOL, "g")
        ps.begin_step()
    ps.capture(steps)
    for _ in range(3):
        ps.g.fill_(float("nan"))
        ps.replay()
        assert_close(host(ps.g), host(want), F32_TOL, "g, replayed")
    ps.begin_step()
    ps.micro_step(steps[0])
    ps.finalize()
    single.begin_step()
    single.micro_step(steps[0])
    assert torch.equal(ps.g, single.g)

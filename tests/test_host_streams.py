"""CPU-only checks of how PrivatiseStep orders its calls: every library call is replaced by a record of the memory it reads and
writes, streams and events by vector clocks, and any two calls that touch the same memory (one of them writing) have to be
ordered by the streams and events they were issued with."""
import contextlib
import gc
import weakref
from dataclasses import replace

import pytest
import torch

import paper_2109_12191_amd as dp
from paper_2109_12191_amd import pipeline
from workloads import conv, get_workload
from workloads.configs import Workload


class _Order:
    """Streams as vector clocks, and every access so far."""

    def __init__(self):
        self.clocks, self.log, self.clashes, self.waits = {}, [], [], set()

    def ring(self, origin: int):
        """Streams other than the origin that have waited for one another, or themselves, in a ring."""
        after = {}
        for waiter, on in self.waits:
            if origin not in (waiter, on):
                after.setdefault(on, set()).add(waiter)
        for s in after:
            seen, todo = set(), set(after[s])
            while todo:
                t = todo.pop()
                seen.add(t)
                todo |= after.get(t, set()) - seen
            if s in seen:
                return s
        return None

    def call(self, stream: int, reads=(), writes=(), what=""):
        clock = self.clocks[stream]
        clock[stream] = clock.get(stream, 0) + 1
        for write, spans in ((False, reads), (True, writes)):
            for a, b in spans:
                for a0, b0, w0, s0, at0, what0 in self.log:
                    if (write or w0) and a < b0 and a0 < b and clock.get(s0, 0) < at0:
                        self.clashes.append((what0, what))
        for write, spans in ((False, reads), (True, writes)):
            self.log += [(a, b, write, stream, clock[stream], what) for a, b in spans]


class _Stream:
    order = None
    count = 0

    def __init__(self, device=None):
        _Stream.count += 1
        self.cuda_stream = _Stream.count
        self.clock = _Stream.order.clocks.setdefault(self.cuda_stream, {})

    def _join(self, other, clock):
        _Stream.order.waits.add((self.cuda_stream, other.cuda_stream))
        for s, at in clock.items():
            self.clock[s] = max(self.clock.get(s, 0), at)

    def wait_stream(self, other):
        self._join(other, other.clock)

    def wait_event(self, event):
        self._join(event.stream, event.clock)


class _Event:
    def record(self, stream):
        self.stream, self.clock = stream, dict(stream.clock)


def _addresses(array):
    return [int(p) if p else 0 for p in array]


@pytest.fixture
def order(monkeypatch):
    dp.load_library()
    o = _Stream.order = _Order()
    main = _Stream()
    o.main = main.cuda_stream
    monkeypatch.setattr(torch.cuda, "Stream", _Stream)
    monkeypatch.setattr(torch.cuda, "Event", _Event)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: main)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)

    def workspaces(bt):
        return [(p, p + b) for p, b in zip(_addresses(bt.ws), bt.ws_bytes)]

    def sizes(bt):
        return [(dp.dp_weight_count(d), dp.dp_bias_count(d)) for d in bt.descs]

    def tables(bt, x, dy, addresses):
        return [(p, p + 8 * bt.descs[0].n) for array in (x, dy) for p in _addresses(array)] if addresses else []

    def per_example(bt, x, dy, g_w, g_b, sqnorm, g_stride=0, stream=None, addresses=False):
        writes = workspaces(bt)                    # (rows of the gradient matrix are stood for by the first one)
        for array, k in ((g_w, 0), (g_b, 1)):
            writes += [(p, p + 4 * s[k]) for p, s in zip(_addresses(array or []), sizes(bt)) if p]
        bt.partial_counts[:] = [1] * bt.n_layers
        o.call(stream, tables(bt, x, dy, addresses), writes, "per_example")

    def unit_grad(bt, unit, x, dy, g_w, g_b, sqnorm, g_stride=0, stream=None, addresses=False):
        per_example(bt, x, dy, g_w, g_b, None, g_stride, stream, addresses)
        o.call(stream, writes=[(p, p + 4 * (bt.descs[0].n // unit)) for p in _addresses(sqnorm)], what="unit norms")

    def norms_from_partials(table, n, n_groups, group_sqnorm, stream=None):
        p = group_sqnorm.data_ptr()
        o.call(stream, [(a, a + 4 * n) for a in _addresses(table.ptrs)], [(p, p + 4 * n_groups * n)], "norms")

    def norms(layer_sqnorm, group_of_layer, n_layers, n, n_groups, group_sqnorm, stream=None):
        p, q = layer_sqnorm.data_ptr(), group_sqnorm.data_ptr()
        o.call(stream, [(p, p + 4 * n_layers * n)], [(q, q + 4 * n_groups * n)], "norms")

    def columns(g, group_sqnorm, n_groups, table, n, run, p, acc, g_stride=0, stream=None):
        g0, q, a0 = g.data_ptr(), group_sqnorm.data_ptr(), acc.data_ptr()
        ends = list(table.begin[1:]) + [p]
        o.call(stream, [(g0, g0 + 4 * p), (q, q + 4 * n_groups * n)],
               [(a0 + 4 * at, a0 + 4 * (at + e - b)) for at, b, e in zip(table.place, table.begin, ends)], "clipped sum, stored")

    def recompute(bt, x, dy, sqnorm, clip_c, acc_w, acc_b, stream=None, addresses=False):
        n = bt.descs[0].n
        acc = [(p, p + 4 * s[k]) for array, k in ((acc_w, 0), (acc_b, 1)) for p, s in zip(_addresses(array), sizes(bt)) if p]
        o.call(stream, [(p, p + 4 * n) for p in _addresses(sqnorm)] + tables(bt, x, dy, addresses), workspaces(bt) + acc, "clipped sum, recomputed")

    def noise(acc, p, *args, step_dev=None, stream=None):
        o.call(stream, writes=[(acc, acc + 4 * p)], what="example noise")

    def finalize(acc, out, *args, stream=None, **kw):
        spans = [(t.data_ptr(), t.data_ptr() + 4 * t.numel()) for t in (acc, out)]
        o.call(main.cuda_stream, spans[:1], spans[1:], "finalize")

    def write_addresses(tensors, example_bytes, n_operands, n_tensors, per_tensor, table, stream=None):
        o.call(main.cuda_stream, writes=[(table, table + 8 * n_operands * n_tensors * per_tensor)], what="addresses")

    for name, fn in dict(dp_per_example_grad_batch=per_example, dp_unit_grad_batch=unit_grad, dp_norms_from_partials=norms_from_partials,
                         dp_norms=norms, dp_clip_accumulate_columns=columns, dp_clip_accumulate_recompute_batch=recompute,
                         dp_add_example_noise=noise, dp_add_noise_finalize_flat=finalize, dp_example_addresses=write_addresses).items():
        monkeypatch.setattr(pipeline.B, name, fn)
    begin = pipeline.PrivatiseStep.begin_step

    def begin_step(self):
        p = self.acc.data_ptr()
        o.call(main.cuda_stream, writes=[(p, p + 4 * self.acc.numel())], what="begin")
        begin(self)

    monkeypatch.setattr(pipeline.PrivatiseStep, "begin_step", begin_step)
    return o


class _Tensor:
    def data_ptr(self):
        return 16


def _steps(wl, count):
    return [[(_Tensor(), _Tensor())] * len(wl.layers)] * count


@pytest.mark.parametrize("noise,unit", [("once", 1), ("per_example", 1), ("once", 2)])
@pytest.mark.parametrize("name,n,hw,sizes", [("resnet18_gn", 24, 40, [6, 5]), ("resnet18_gn", 32, 24, [6, 5]), ("resnet50", 16, 64, [3, 3, 2]),
                                             ("resnet50_nano", 1, 64, [3, 2, 2]), ("resnet20", 8, 32, [2, 2, 1]), ("resnet20", 8, 32, [5])])
def test_calls_on_the_same_memory_are_ordered_when_phases_differ(order, monkeypatch, name, n, hw, sizes, noise, unit):
    """Plans of different size deal the layers to the streams differently: a tensor's clipped sums stay in order all the same, and
    so do the buffers."""
    if n % unit:
        pytest.skip("units of two examples need an even micro-step")
    monkeypatch.setattr(pipeline.PrivatiseStep, "_micro_steps_together", lambda self: sizes[0])
    wl = get_workload(name, n=n, accum=sum(sizes), hw=hw)
    ps = dp.PrivatiseStep(wl, device="cpu", streams=8, noise=noise, clip_unit=unit)
    assert ps._phase_sizes(sum(sizes)) == sizes
    for _ in range(2):
        ps.run(_steps(wl, sum(sizes)))
    ps.begin_step()
    for inputs in _steps(wl, 3):                  # micro-steps one by one between whole steps
        ps.micro_step(inputs)
    ps.finalize()
    ps.run(_steps(wl, sum(sizes)))
    ps.run(_steps(wl, 2 * sum(sizes) - 1))        # a step of another length
    assert not order.clashes, (len(order.clashes), order.clashes[:4])
    # a stream capture joins the side streams by their waits: none may hang on itself
    assert order.ring(order.main) is None


class _Graph:
    pass


def test_a_recorded_step_keeps_its_example_addresses(order, monkeypatch):
    """Two graphs of one PrivatiseStep, and a graph that the caller records: none reads or writes addresses that were given away."""
    capturing = [False]

    @contextlib.contextmanager
    def graph(g):
        capturing[0] = True
        yield
        capturing[0] = False

    monkeypatch.setattr(torch.cuda, "CUDAGraph", _Graph)
    monkeypatch.setattr(torch.cuda, "graph", graph)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: capturing[0])
    tables, write = [], pipeline.B.dp_example_addresses

    def seen(tensors, example_bytes, n_operands, n_tensors, per_tensor, table, stream=None):
        tables.append(table)
        write(tensors, example_bytes, n_operands, n_tensors, per_tensor, table, stream)

    monkeypatch.setattr(pipeline.B, "dp_example_addresses", seen)
    wl = get_workload("resnet18_gn", n=2, accum=3, hw=16)
    ps = dp.PrivatiseStep(wl, device="cpu")
    graphs = [ps.capture(_steps(wl, 3)) for _ in range(2)]
    kept = [weakref.ref(g.example_addresses) for g in graphs]
    assert kept[0]().data_ptr() != kept[1]().data_ptr() and {k().data_ptr() for k in kept} <= set(tables)
    with graph(None):
        ps.run(_steps(wl, 3))
    recorded = tables[-1]
    for count in (3, 5, 2):                       # (a longer step needs a larger table)
        ps.run(_steps(wl, count))
        assert tables[-1] not in [recorded] + [k().data_ptr() for k in kept]
    with graph(None):
        ps.run(_steps(wl, 3))
    assert tables[-1] != recorded
    del graphs[0]
    gc.collect()
    assert kept[0]() is None and kept[1]() is not None


def test_steps_on_another_stream_get_addresses_of_their_own(order, monkeypatch):
    """A table is used again only on the stream on which its readers were waited for."""
    wl = get_workload("resnet18_gn", n=2, accum=3, hw=16)
    ps = dp.PrivatiseStep(wl, device="cpu")
    ps.run(_steps(wl, 3))
    first = ps._addresses[1]
    ps.run(_steps(wl, 3))
    assert ps._addresses[1] is first
    other = _Stream()
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: other)
    ps.run(_steps(wl, 3))
    assert ps._addresses[1] is not first


def test_buffers_do_not_grow_with_the_lengths_of_the_steps(order):
    """Steps of every length run in the buffers of the first; a smaller phase uses the front of them."""
    wl = get_workload("resnet50_nano", accum=16, hw=64)
    ps = dp.PrivatiseStep(wl, device="cpu", streams=4)

    def held():
        tensors = [t for o in gc.get_objects() if type(o) is pipeline._Store for t in (o.g, o.ws, o.group_sqnorm, o.layer_sqnorm) if t is not None]
        return sum(t.numel() * t.element_size() for t in tensors)

    ps.run(_steps(wl, 16))
    gc.collect()
    before = held()
    ps.begin_step()
    ps.micro_step(_steps(wl, 1)[0])               # one at a time: the second copy, of a micro-step
    ps.finalize()
    one = 4 * ps.p_mat + sum(ps._plan(1).ws_bytes) + (1 << 20)
    for count in (1, 2, 3, 7, 11, 15, 16, 17, 29):
        ps.run(_steps(wl, count))
    assert before <= held() <= before + one
    assert not order.clashes
    for plan in ps._plans.values():
        for c, store in enumerate(plan.stores):
            assert plan.rows <= store.rows and plan.ws[c][-1] + plan.ws_bytes[-1] <= store.ws.data_ptr() + store.ws.numel()
            assert plan.g[c].data_ptr() == store.g.data_ptr()


@pytest.mark.parametrize("name,n,accum,mode,streams", [("resnet18_gn", 4, 64, "materialise", 8), ("resnet50_nano", 1, 1024, "auto", 4),
                                                       ("resnet50", 2, 64, "auto", 1), ("resnet20", 3, 80, "recompute", 2)])
def test_a_phase_is_bounded_by_what_it_holds(order, monkeypatch, name, n, accum, mode, streams):
    """Gradients, norms and workspaces of all copies stay within the bound, whatever the inputs weigh; one micro-step always goes."""
    wl = get_workload(name, n=n, accum=accum, hw=64 if name != "resnet20" else 32)
    for bound in (pipeline.PHASE_STORE_BYTES, 1e9, 1.0):
        monkeypatch.setattr(pipeline, "PHASE_STORE_BYTES", bound)
        ps = dp.PrivatiseStep(wl, device="cpu", mode=mode, streams=streams)
        size, copies = ps.micro_steps_per_phase, len(ps._main.stores)
        assert size == 1 or copies * (4 * ps._main.rows * ps.p_mat + ps._workspace_bytes(size)) <= bound
        assert copies == (ps.copies if size == 1 or accum > size else 1)


# micro-steps per phase on both sides of the lines that decide it
@pytest.mark.parametrize("name,n,accum,hw,want", [
    ("resnet50", 28, 4, 224, 4), ("resnet50", 32, 4, 224, 1), ("resnet50", 40, 4, 192, 1), ("resnet50", 16, 8, 224, 4), ("resnet50", 40, 4, 160, 2),
    ("resnet20", 64, 4, 32, 4), ("resnet20", 128, 4, 32, 2), ("resnet20", 256, 4, 32, 1), ("resnet18_gn", 64, 8, 32, 4),
    ("resnet18_gn", 24, 8, 40, 4), ("resnet18_gn", 48, 4, 40, 2), ("resnet18_gn", 64, 4, 40, 1), ("resnet18_gn", 96, 4, 24, 1),
    ("resnet50_nano", 1, 64, 224, 64), ("resnet50_nano", 1, 1024, 224, 47), ("resnet18_gn f32", 10, 4, 40, 4)])
def test_micro_steps_per_phase(order, name, n, accum, hw, want):
    name, *dtype = name.split()
    wl = get_workload(name, n=n, accum=accum, hw=hw)
    wl = replace(wl, dtype=dtype[0] if dtype else wl.dtype)
    ps = dp.PrivatiseStep(wl, device="cpu", streams=8)
    size = ps.micro_steps_per_phase
    assert size == want and ps._phase_sizes(accum)[0] == size
    alone, together = ps._gathers(1), ps._gathers(size)
    assert not any(now and not before for now, before in zip(together, alone))      # no layer loses its kernel


def test_micro_steps_from_a_generator_are_taken_one_by_one(order, monkeypatch):
    """run() takes any iterable; one that is no list may hand over the same tensors again and again, so nothing is read ahead."""
    wl = get_workload("resnet20", n=4, accum=5, hw=32)
    ps = dp.PrivatiseStep(wl, device="cpu")
    assert ps.micro_steps_per_phase == 5
    seen = []
    call = pipeline.B.dp_norms_from_partials
    monkeypatch.setattr(pipeline.B, "dp_norms_from_partials", lambda *a, **k: (seen.append("issued"), call(*a, **k)))

    def micro_steps():
        for _ in range(5):
            seen.append("made")
            # (an entry may say more than (x, dy), and layers may be looked up by number)
            yield {i: (_Tensor(), _Tensor(), "more") for i in range(len(wl.layers))}

    ps.run(micro_steps())
    assert seen == ["made", "issued"] * 5 and ps.micro_steps_done == 5
    del seen[:]
    ps.run(tuple(_steps(wl, 5)))
    assert seen == ["issued"]


@pytest.mark.parametrize("streams", [1, 4])
def test_what_a_step_shows_is_one_micro_steps(order, streams):
    """Norms, rows and work are those of a micro-step, the norms a matrix of their own, however many micro-steps share a phase."""
    wl = get_workload("resnet50_nano", accum=8, hw=64)
    ps = dp.PrivatiseStep(wl, device="cpu", streams=streams)
    assert ps.micro_steps_per_phase == 8 and ps.rows == 1 and ps.work[0][0] == wl.layers[0].flops and ps.descs[0].n == 1
    for run in (lambda: ps.run(_steps(wl, 8)), lambda: ps.micro_step(_steps(wl, 1)[0]), lambda: ps.run(_steps(wl, 3))):
        run()
        assert ps.group_sqnorm.shape == (wl.n_groups, 1) and ps.group_sqnorm.is_contiguous() and ps.g.shape == (1, ps.p_mat)
    # and of the last micro-step of the last phase
    ps._plan(8).group_sqnorm[0].copy_(torch.arange(wl.n_groups * 8, dtype=torch.float32).view(wl.n_groups, 8))
    ps.run(_steps(wl, 8))
    assert torch.equal(ps.group_sqnorm[:, 0], torch.arange(wl.n_groups, dtype=torch.float32) * 8 + 7)
    # as many of the last micro-steps' norms as there are buffer copies, by the number of the micro-step
    for m in range(8 - ps.copies, 8):
        assert torch.equal(ps._group_sqnorm[m % ps.copies][:, 0], torch.arange(wl.n_groups, dtype=torch.float32) * 8 + m)


def test_buffers_go_with_their_step(order):
    """Nothing keeps a PrivatiseStep that was dropped: its memory is given back at once, not when cycles are next collected."""
    gc.collect()
    gc.disable()
    try:
        ps = dp.PrivatiseStep(get_workload("resnet18_gn", n=2, accum=3, hw=16), device="cpu", streams=4)
        ps.run(_steps(ps.wl, 3))
        ps.begin_step()
        ps.micro_step(_steps(ps.wl, 1)[0])
        ps.finalize()
        kept = [weakref.ref(o) for o in [ps] + [st for st in ps._stores if st is not None] + list(ps._plans.values())]
        assert len(kept) == 5
        del ps
        assert all(k() is None for k in kept)
    finally:
        gc.enable()


@pytest.mark.parametrize("n,accum,hw,streams", [(1, 64, 224, 4), (1, 3, 224, 1), (2, 16, 192, 4), (1, 24, 160, 1), (1, 8, 64, 4)])
def test_workspaces_in_the_gradient_matrix_lie_behind_the_stored_columns(order, n, accum, hw, streams):
    """A phase that recomputes keeps the stored columns side by side at the front of the matrix and the workspaces of the other layers in
    the rest of it, each to itself; what it stores goes to the accumulator's places."""
    wl = get_workload("resnet50_nano", n=n, accum=accum, hw=hw)
    ps = dp.PrivatiseStep(wl, device="cpu", streams=streams)
    for tensors in {accum, max(2, accum // 2), 3}:
        plan, inside = ps._plan(tensors), ps._in_matrix(tensors)
        if n * tensors < 3:
            assert plan.form is ps.form
            continue
        assert plan.form.count("recompute") >= 10 and all(l.kind == "dense" for l, f, k in zip(ps.layers, plan.form, inside) if f == "recompute" and not k)
        for c, store in enumerate(plan.stores):
            first, end = store.g.data_ptr() + 4 * plan.rows * plan.p_mat, store.g.data_ptr() + 4 * store.g.numel()
            spans = sorted((at, at + b) for at, b, k in zip(plan.ws[c], plan.ws_bytes, inside) if k)
            assert first <= spans[0][0] and spans[-1][1] <= end and all(a[1] <= b[0] for a, b in zip(spans, spans[1:]))
            rest = [(at, at + b) for at, b, k in zip(plan.ws[c], plan.ws_bytes, inside) if not k]
            assert store.ws.data_ptr() <= min(rest)[0] and max(rest)[1] <= store.ws.data_ptr() + store.ws.numel()
        ends = list(plan.segments.begin[1:]) + [plan.p_mat]
        for i, form in enumerate(plan.form):
            if form == "materialise":
                k = max(s for s in range(plan.segments.n_seg) if plan.segments.begin[s] <= plan.off_w[i])
                assert plan.off_w[i] + ps.pw[i] <= ends[k] and plan.segments.group[k] == ps.group_of_layer[i]
                assert plan.segments.place[k] + plan.off_w[i] - plan.segments.begin[k] == ps.off_w[i]


@pytest.mark.parametrize("streams,sizes", [(1, [8]), (4, [8]), (4, [5, 4])])
def test_last_gradients_that_a_phase_does_not_store_are_stored_apart(order, monkeypatch, streams, sizes):
    """Every layer's gradients of the last micro-step are written once, into a matrix that nothing else of the step uses, and the end of the
    step waits for them; earlier phases write none."""
    monkeypatch.setattr(pipeline.PrivatiseStep, "_micro_steps_together", lambda self: sizes[0])
    wl = get_workload("resnet50_nano", accum=sum(sizes), hw=64)
    ps = dp.PrivatiseStep(wl, device="cpu", streams=streams)
    writes, call = [], pipeline.B.dp_per_example_grad_batch

    def seen(bt, x, dy, g_w, *rest, **kw):
        writes.extend(p for p in _addresses(g_w or []) if p)
        call(bt, x, dy, g_w, *rest, **kw)

    monkeypatch.setattr(pipeline.B, "dp_per_example_grad_batch", seen)
    for _ in range(2):
        del writes[:]
        ps.run(_steps(wl, sum(sizes)))
        apart = ps._last_store.g
        for i, form in enumerate(ps._plan(sizes[-1]).form):
            assert writes.count(apart.data_ptr() + 4 * ps.off_w[i]) == (form == "recompute")
        order.call(order.main, [(apart.data_ptr(), apart.data_ptr() + 4 * apart.numel())], what="a reader")
    assert ps.g.data_ptr() == apart.data_ptr() and ps.g.shape == (1, ps.p_mat)
    assert not order.clashes and order.ring(order.main) is None


def _rows_workload(n, accum):
    """Two layers whose gradients phases that others follow do not store, one whose they do."""
    layers = (conv(1024, 256, 1, 1, 14, name="a"), conv(64, 64, 3, 1, 14, name="b"), conv(256, 1024, 1, 1, 14, name="c"))
    return Workload("rows", layers, n, accum, "bf16", "per_layer", 1.0, 0.0, ("abs",) * 3, 0.01, 77)


@pytest.mark.parametrize("noise", ["once", "per_example"])
@pytest.mark.parametrize("sizes,streams", [([1, 1, 1], 8), ([2, 2, 1], 8), ([3, 2], 3), ([2, 2, 1], 1)])
def test_calls_are_ordered_where_phases_that_others_follow_store_less(order, monkeypatch, sizes, streams, noise):
    """The last phase's plan is another one, of another division of the matrix; steps of another length and single micro-steps in between."""
    monkeypatch.setattr(pipeline.PrivatiseStep, "_micro_steps_together", lambda self: sizes[0])
    wl = _rows_workload(140, sum(sizes))
    ps = dp.PrivatiseStep(wl, device="cpu", streams=streams, noise=noise)
    lean, last = ps._plan(sizes[0], True), ps._plan(sizes[-1])
    assert lean.form == ["recompute", "materialise", "recompute"] and last.form is ps.form and lean.p_mat < last.p_mat == ps.p_mat
    for steps in (sum(sizes), sum(sizes), 1, 2 * sum(sizes) - 1):
        ps.run(_steps(wl, steps))
        assert ps._g_plan.form is ps.form and ps.micro_steps_done == steps
    ps.begin_step()
    for inputs in _steps(wl, 3):
        ps.micro_step(inputs)
    ps.finalize()
    ps.run(_steps(wl, sum(sizes)))
    assert not order.clashes, (len(order.clashes), order.clashes[:4])
    assert order.ring(order.main) is None


@pytest.mark.parametrize("streams", [1, 4])
@pytest.mark.parametrize("name,sizes,phase", [("rows", [1, 1, 1], 2), ("rows", [2, 2, 1], 1), ("resnet50_nano", [5, 4], 1)])
def test_a_step_that_is_broken_off_leaves_the_last_gradients_whole(order, monkeypatch, name, sizes, phase, streams):
    """What the last phase before that did not store is stored then, apart, and the current stream comes after it."""
    monkeypatch.setattr(pipeline.PrivatiseStep, "_micro_steps_together", lambda self: sizes[0])
    wl = _rows_workload(140, sum(sizes)) if name == "rows" else get_workload(name, accum=sum(sizes), hw=64)
    ps = dp.PrivatiseStep(wl, device="cpu", streams=streams)
    norms, writes, call = [], [], pipeline.B.dp_per_example_grad_batch

    def broken(*args, **kw):
        norms.append(1)
        if len(norms) > phase:
            raise KeyboardInterrupt

    def seen(bt, x, dy, g_w, *rest, **kw):
        writes.extend(p for p in _addresses(g_w or []) if p)
        call(bt, x, dy, g_w, *rest, **kw)

    monkeypatch.setattr(pipeline.B, "dp_norms_from_partials", broken)
    monkeypatch.setattr(pipeline.B, "dp_per_example_grad_batch", seen)
    with pytest.raises(KeyboardInterrupt):
        ps.run(_steps(wl, sum(sizes)))
    apart, form = ps._last_store.g, ps._plan(sizes[phase - 1], True).form
    assert form.count("recompute") >= 2
    for i, f in enumerate(form):
        assert writes.count(apart.data_ptr() + 4 * ps.off_w[i]) == (f != ps.form[i])
    order.call(order.main, [(apart.data_ptr(), apart.data_ptr() + 4 * apart.numel())], what="a reader")
    assert ps.g.data_ptr() == apart.data_ptr() and ps.g.shape == (ps.rows, ps.p_mat) and ps._not_stored is None

"""Sequencing of the C-ABI calls for one optimiser step of a layer set.

This class owns device buffers (allocated through torch) and issues the library calls in
order; it performs no arithmetic of its own.  Per micro-step:
    dp_per_example_grad_batch (one call per group of layers that run the same kernel)  ->  dp_norms_from_partials  ->
    dp_clip_accumulate_columns (materialised layers) and dp_clip_accumulate_recompute_batch (the rest);
once per optimiser step: dp_add_noise_finalize_flat over all parameter tensors.

`run` and `capture` see the micro-steps of a whole step at once and issue several of them together where they are small:
every example is still clipped by its own norms, but the launches hold the examples of all of them (the "_at" calls, whose
operands are arrays of example addresses), the clipped sum reads and writes the accumulator once, and a step of 64
one-example micro-steps is two dozen launches instead of a thousand.

Each layer uses one of the two forms of the clipped sum.  "materialise" keeps the layer's
per-example gradients of the micro-step in a [n, P] matrix (written by the contraction's
epilogue, read once by the streaming accumulate); "recompute" keeps nothing and runs a
second, clip-factor-weighted contraction.  `mode="auto"` picks per layer whichever moves
fewer bytes / flops; early conv layers (few parameters, large feature maps) materialise,
late ones (many parameters, tiny feature maps) recompute.
"""
from __future__ import annotations

from typing import Iterable, List, Optional, Sequence

import torch

from . import binding as B

# Which micro-steps are issued together (a phase): it saves launches and fills the chip where a micro-step is small.  MI355X, us per
# step of four micro-steps on eight streams, one by one / in phases, on both sides of each line:
#   a micro-step that reads more than this fills the chip by itself.  ResNet-50 with 24 examples (1.05 GB) 3141 / 2999, 28 (1.22 GB)
#   3613 / 3500; 32 (1.39 GB) 3853 / 3999, 40 (1.74 GB) 4656 / 4927; at 192 x 192, 40 examples (1.28 GB) 5013 / 5245
PHASE_MICRO_STEP_BYTES = 1.25e9
#   examples of a phase.  ResNet-20, 64 examples a micro-step: phases of 128 / 256 784 / 667; ResNet-18-GN, 48 (8 micro-steps): one by
#   one / 192 2840 / 2470, 64: one by one / 256 3452 / 3223 (128: 6101 / 6338, a loss inside the line).  Beyond, ResNet-20, 256: one by one /
#   512 2493 / 2411; ResNet-18-GN, 48: 192 / 384 2470 / 2556, 64: 256 / 512 3223 / 7084
PHASE_EXAMPLES = 256
#   and of micro-steps of one or two examples.  ResNet-50, 64 x 1: one by one / 16 / 32 / 64 9682 / 2774 / 2476 / 2481; 32 x 2: 7984 /
#   2821 (16) / 2502 / 2498
PHASE_EXAMPLES_OF_SMALL = 64
# How much work a batch call needs for its clip-weighted layers on 14 x 14 maps to gain by the whole-row kernel (from finished fp32 blocks) so much that they need no
# stored gradients, in rounds of 768 workgroups of one 128 x 128 x 64 chunk, with seventeen examples (two ranges) and more / with twelve.
# Us a step, stored / this: six layers of 256 -> 256, six micro-steps of 110 examples (10.5) 624 / 479 on three streams; 256 -> 256 and 1024 -> 256, 130 examples (10.4) 644 / 545;
# those beside a 3x3 and other layers 1258 / 1216 on three streams, 1195 / 1300 on eight, with 64 examples (5.1) 542 / 548.  ResNet-50 in phases of
# one-example micro-steps on four streams: 16 examples (13) 708 / 720, 18 (14, on one) 953 / 933, 20 (16) 902 / 873, 24 (19, of two on one stream) 1173 / 1157,
# 32 (26) 1150 / 1111, 64 (53) 2140 / 2050.
ROWS_WORK = 10, 17
# And no phase is so large that a layer falls back to the kernel that gathers its operands element by element, because the rewritten
# operands of a faster one outgrow their share of the workspace: ResNet-18-GN at 40 x 40, 64 examples 3656 / 5083 (two micro-steps) / 7188
# (four), 24 (8 micro-steps): 3097 / 3028 (four) / 3825 (eight).
# What a phase may hold in stored gradients, norms and workspaces, all copies together (4 % of the card's memory); a single
# micro-step takes what it needs.
PHASE_STORE_BYTES = 12e9


def _pad4(v: int) -> int:
    return (v + 3) & ~3


def _align256(v: int) -> int:
    return (v + 255) & ~255


class _Store:
    """One copy of what a phase writes before its clipped sum is done: the gradient matrix, the norms and the workspaces.  The plans
    of all phase sizes share it (a smaller phase uses the front of every buffer)."""

    def __init__(self, ps: "PrivatiseStep", rows: int, ws_bytes: int):
        dev, f32 = ps.device, torch.float32
        self.rows, self.ws_bytes = rows, ws_bytes
        self.g = torch.empty((rows, ps.p_mat), dtype=f32, device=dev) if ps.p_mat else None
        if self.g is not None:                     # the columns between tensors are read by the clipped sum, never written
            for i, form in enumerate(ps.form):
                if form == "materialise":
                    for col, size in ((ps.off_w[i], ps.pw[i]), (ps.off_b[i], ps.pb[i])):
                        if size % 4:
                            self.g[:, col + size: col + _pad4(size)] = 0.0
        self.group_sqnorm = torch.zeros(ps.n_groups * rows, dtype=f32, device=dev)
        self.layer_sqnorm = torch.zeros(len(ps.layers) * rows, dtype=f32, device=dev) if ps.clip_unit > 1 else None
        self.ws = torch.empty(ws_bytes, dtype=torch.uint8, device=dev)
        self.done = None                           # events after which its buffers are free again


class _Plan:
    """Views and batch calls for phases of `n` examples: one micro-step in the caller's tensors (`tensors` = 1), or `tensors`
    micro-steps through arrays of example addresses.  `only`: per-example calls of these layers and nothing else.  (Keeps no reference to its
    PrivatiseStep: the buffers go when that goes.)"""

    def __init__(self, ps: "PrivatiseStep", tensors: int, stores: List[_Store], only: Optional[Sequence[int]] = None, more: bool = False):
        wl = ps.wl
        self.tensors = tensors
        self.stores = stores                       # the copies that are large enough
        self.n = wl.n * tensors
        self.rows = self.n // ps.clip_unit
        self.layers = ps.layers
        self.form = ps._forms(tensors, more)
        self.blocks = ps._blocks(tensors)
        L = len(self.layers)
        self.descs, need = ps._workspaces(tensors)
        self.g = [st.g[: self.rows] if st.g is not None else None for st in stores]
        self.off_w, self.off_b, self.p_mat = ps.off_w, ps.off_b, ps.p_mat
        free = [None] * len(stores)
        if self.form is not ps.form:
            # only some of the layers that the matrix has columns for are stored: their columns move together, and what is left of
            # the matrix holds the workspaces of the others
            self.off_w, self.off_b, self.p_mat = ps._columns(self.form)
            free = [g.data_ptr() + 4 * self.rows * self.p_mat for g in self.g]
            self.g = [g.view(-1)[: self.rows * self.p_mat].view(self.rows, self.p_mat) for g in self.g]
        self.group_sqnorm = [st.group_sqnorm[: ps.n_groups * self.rows].view(ps.n_groups, self.rows) for st in stores]
        self.layer_sqnorm = [st.layer_sqnorm[: L * self.rows].view(L, self.rows) for st in stores] if ps.clip_unit > 1 else None
        self.segments = ps._segments(self.form, self.off_w) if self.p_mat else None
        # a workspace per layer (the layers of a phase are in flight together)
        self.ws_bytes = need
        self.ws = []
        for st, spare in zip(stores, free):
            at, spare, where = st.ws.data_ptr(), spare and _align256(spare), []
            for b, inside in zip(need, ps._in_matrix(tensors) if self.blocks else [False] * L):
                where.append(spare if inside else at)
                if inside:
                    spare += _align256(b)
                else:
                    at += _align256(b)
            self.ws.append(where)
        # Layers that run the same kernel variant go to the library in ONE batch call, which puts them into one
        # launch (at most 16 per launch): per phase a micro-step is a dozen launches, not a hundred.
        self.variant = [(B.dp_kernel_variant(d, B.DP_WS_PER_EXAMPLE_GRAD | self.blocks | B.DP_VARIANT_SHARED |
                                             (B.DP_VARIANT_MATERIALISE if form == "materialise" else 0)),
                         B.dp_kernel_variant(d, B.DP_WS_RECOMPUTE | self.blocks | B.DP_VARIANT_SHARED) if form == "recompute" else "")
                        for d, form in zip(self.descs, self.form)]
        self.partials = [B.PartialTable(self.ws[c], [1] * L, ps.group_of_layer)
                         for c in range(len(stores))]
        self.work = ps._work(tensors, more)
        self.groups_a = self._make_groups(ps, range(L) if only is None else only, 0) if ps.clip_unit == 1 else []
        self.groups_b = self._make_groups(ps, [i for i in range(L) if self.form[i] == "recompute"], 1) if only is None else []
        self.groups_u = self._make_groups(ps, range(L), 2) if ps.clip_unit > 1 else []

    def _make_groups(self, ps: "PrivatiseStep", layer_ids, use: int):
        """Groups of at most 16 layers with the same kernel variant for phase `use` (0: per-example gradients,
        1: recomputing clipped sum, 2: unit sums), largest total work first.  Each group: dict(layers, name, batch per copy,
        constant pointer arrays)."""
        by_name = {}
        family = "conv3x3_rows<bf16,all widths,%s>" % ("weighted" if use == 1 else "per_example")
        for li in layer_ids:
            key = self.variant[li][1 if use == 1 else 0]      # same name, same kernel
            if ps.batching == "all":
                key = "all layers"
            elif key.startswith("conv3x3_rows<"):
                # inside a batch call the library runs all variants of the raw-row 3x3 kernel in one launch (only
                # four kernels run at a time on the chip: the few workgroups of a narrow layer cost none of the
                # four inside a wide launch), so the family is one batch call
                key = family
            by_name.setdefault(key, []).append(li)
        groups = []
        for key, ids in by_name.items():
            width = len(ids) if (ps.batching == "all" or key == family) else 16
            for k in range(0, len(ids), width):
                part = ids[k: k + width]
                name = key
                if len(part) == 1:           # a single layer is planned as a launch of its own
                    name = B.dp_kernel_variant(self.descs[part[0]], self.blocks | (B.DP_WS_RECOMPUTE if use == 1 else (
                        B.DP_WS_PER_EXAMPLE_GRAD | (B.DP_VARIANT_MATERIALISE if self.form[part[0]] == "materialise" else 0))))
                g = dict(layers=part, name=name, conv=all(self.layers[i].kind == "conv" for i in part))
                g["batch"] = [B.LayerBatch([self.descs[i] for i in part], [self.ws[c][i] for i in part],
                                           [self.ws_bytes[i] for i in part], bool(self.blocks))
                              for c in range(len(self.stores))]
                if use == 2:
                    g["usq"] = [g["batch"][c].ptrs([self.layer_sqnorm[c][i].data_ptr() for i in part])
                                for c in range(len(self.stores))]
                if use != 1:
                    g["counted"] = False
                    mat = [self.form[i] == "materialise" for i in part]
                    g0 = [g.data_ptr() if g is not None else 0 for g in self.g]
                    g["gw"] = [g["batch"][c].ptrs([g0[c] + 4 * self.off_w[i] if m else None
                                                   for i, m in zip(part, mat)]) if any(mat) else None for c in range(len(self.stores))]
                    g["gb"] = [g["batch"][c].ptrs([g0[c] + 4 * self.off_b[i] if (m and ps.pb[i]) else None
                                                   for i, m in zip(part, mat)]) if any(mat) else None for c in range(len(self.stores))]
                else:
                    acc0 = ps.acc.data_ptr()
                    g["sq"] = [g["batch"][c].ptrs([self.group_sqnorm[c][ps.group_of_layer[i]].data_ptr() for i in part])
                               for c in range(len(self.stores))]
                    g["clip"] = g["batch"][0].floats([ps.group_clip[ps.group_of_layer[i]] for i in part])
                    g["acc_w"] = g["batch"][0].ptrs([acc0 + 4 * ps.off_w[i] for i in part])
                    g["acc_b"] = g["batch"][0].ptrs([acc0 + 4 * ps.off_b[i] if ps.pb[i] else None
                                                     for i in part])
                g["flops"] = sum(self.layers[i].flops for i in part) * self.n
                g["bytes"] = sum(self.work[i][2 if use == 1 else 1] for i in part)
                g["seconds"] = self._estimate(ps, g)
                groups.append(g)
        groups.sort(key=lambda g: -g["seconds"])
        # side stream of each group: longest first onto the least loaded stream
        load = [0.0] * max(1, ps.n_streams)
        for gi, g in enumerate(groups):
            k = load.index(min(load)) if ps.lanes != "round_robin" else gi % max(1, ps.n_streams)
            g["lane"] = k
            load[k] += g["seconds"]
        return groups

    def _estimate(self, ps: "PrivatiseStep", g) -> float:
        """Duration of a group's launch for the lane balance: its work at the rates its kernel family sustains on
        MI355X when it has the chip to itself (measured call by call on ResNet-50 at n = 32), plus a few
        microseconds per launch however small it is."""
        if ps.lanes == "flops" or self.n <= 2:
            # micro-steps of one or two examples: launches are bound by the walk along K of a few workgroups, not by
            # the chip's rates; flops alone order them better (measured: 5.6 k against 5.1 k examples/s)
            return g["flops"] / 150.0e12 + 8.0e-6
        name = g["name"]
        if name.startswith("conv3x3_rows"):
            rate = 300.0e12                      # (100 .. 300: the same step time; the family is one launch per phase)
        elif "gather" in name:
            rate = 130.0e12
        else:
            rate = 400.0e12
        return max(g["flops"] / rate, g["bytes"] / 4.5e12) + 8.0e-6


class PrivatiseStep:
    def __init__(self, wl, device: str = "cuda:0", mode: str = "auto", streams: int = 1, noise: str = "once",
                 batching: str = "variant", lanes: str = "balanced", clip_unit: int = 1, fork: Optional[str] = None):
        B.load_library()
        self.wl = wl
        if batching not in ("variant", "all"):
            raise ValueError(batching)
        # "variant": one batch call per kernel variant, spread over the side streams (large micro-batches: the
        # launches are long and overlap); "all": one batch call per phase with every layer in it, so that also the
        # pre-passes and slice sums of all layers share launches (one-example micro-steps: launches are what costs)
        self.batching = batching
        if lanes not in ("round_robin", "balanced", "flops"):
            raise ValueError(lanes)
        self.lanes = lanes                     # how the batch calls of a phase are dealt to the side streams
        # "micro_step": the side streams of the per-example phase start every micro-step behind everything issued so
        # far; "step": only the first micro-step of a step does -- later ones follow their own stream's previous
        # micro-step (and the clipped sum that last read their buffer copy), so they overlap the norm launches and the
        # clipped sum of the micro-step before.  Worth it when the launches are short (phases of one or two examples).
        if fork not in (None, "micro_step", "step"):
            raise ValueError(fork)
        self.fork = fork
        if noise not in ("once", "per_example"):
            raise ValueError(noise)
        # "once": N(0, sigma^2 C^2) added in finalize (first equation of the Algorithm section);
        # "per_example": every clipped example brings N(0, sigma^2 C^2 / |B|) (second equation)
        self.noise = noise
        self.device = torch.device(device)
        self.layers = list(wl.layers)
        self.n = wl.n
        # Clipping units of several consecutive examples (the micro-batching of the GPU baseline, Abstract and
        # Table 1): the path runs on the unit SUMS with every bound multiplied by the unit size, which gives
        # (noise + sum of the clipped unit means) / (number of units); a unit is one row wherever an example is.
        self.clip_unit = int(clip_unit)
        if self.clip_unit < 1 or wl.n % self.clip_unit:
            raise ValueError("the micro-step size must be a multiple of clip_unit")
        if self.clip_unit > 1 and noise != "once":
            raise ValueError("per-example noise is defined for units of one example")
        self.rows = wl.n // self.clip_unit         # of a micro-step
        L = len(self.layers)
        descs = [B.make_desc(l, wl.n, wl.dtype) for l in self.layers]
        self.pw = [B.dp_weight_count(d) for d in descs]
        self.pb = [B.dp_bias_count(d) for d in descs]
        self.group_of_layer = list(wl.group_of_layer)
        self.group_clip, self.clip_total = B.dp_group_clip_bounds(wl.clip_c, wl.n_groups)
        if self.clip_unit > 1:
            self.group_clip = [c * self.clip_unit for c in self.group_clip]
            self.clip_total *= self.clip_unit
            mode = "materialise"                   # the unit sums are 1/unit of the per-example matrix: keep them
        self._mode = mode
        self.n_groups = wl.n_groups

        self.form = [self._choose(l, mode, wl.n) for l in self.layers]

        # flat parameter vector: materialised layers first (their columns double as the
        # layout of the per-example gradient matrix), then the recomputed ones
        mat = [i for i in range(L) if self.form[i] == "materialise"]
        self.off_w = [0] * L
        self.off_b = [0] * L
        pos = 0
        self.p_mat = 0
        for i in mat + [i for i in range(L) if self.form[i] == "recompute"]:
            self.off_w[i] = pos
            pos += _pad4(self.pw[i])
            self.off_b[i] = pos
            pos += _pad4(self.pb[i])
            if self.form[i] == "materialise":
                self.p_mat = pos
        self.p_total = max(pos, 4)
        # every tensor of the flat vector with its Philox tensor id (2*layer weight, 2*layer+1 bias), in
        # the order they lie in memory: the table of the one-launch finalize
        tensors = sorted([(self.off_w[i], self.pw[i], 2 * i) for i in range(L)] +
                         [(self.off_b[i], self.pb[i], 2 * i + 1) for i in range(L) if self.pb[i]])
        self._tensors = B.TensorTable([t[0] for t in tensors], [t[1] for t in tensors], [t[2] for t in tensors])
        dev = self.device
        f32 = torch.float32
        self.acc = torch.zeros(self.p_total, dtype=f32, device=dev)
        self.out = torch.zeros(self.p_total, dtype=f32, device=dev)
        # Workspaces and per-phase buffers (_Store).  With one stream all calls run in order and share
        # one copy.  With side streams the layers of a phase run concurrently and the per-example part of a phase overlaps the
        # clipped sum of the one before: everything a phase writes before its clipped sum is done -- the gradient matrix, the
        # norms, the workspaces -- exists twice and phases alternate between the copies.
        self.n_streams = max(1, int(streams))
        self.copies = 2 if self.n_streams > 1 else 1
        self.group_of_layer_dev = torch.tensor(self.group_of_layer, dtype=torch.int32, device=dev)
        esize = 2 if wl.dtype == "bf16" else 4
        self._example_bytes = [b for l in self.layers for b in (l.x_bytes(esize), l.dy_bytes(esize))]
        self._last_store = None                  # gradients of a last micro-step that its phase does not store (_last_plan)
        self._last_plans = {}
        self._phase_forms = {}                   # micro-steps of a phase -> forms of the layers
        self._lean_forms = {}                    # and of one that others follow
        self._inside = {}                        # and whose workspaces lie in the gradient matrix
        self._ws_bytes = {}                      # and how much the others take together
        self._needs = {}                         # micro-steps of a phase -> descriptors and workspace sizes
        self._together = self._micro_steps_together()
        # Micro-steps that a copy has room for.  A step of one phase never uses a second copy; micro-steps that are handed over
        # one by one do.  Steps of more micro-steps than the workload's have more phases, not larger ones.
        self._ws_room = None
        sizes = self._phase_sizes(max(1, wl.accum))
        self._ws_room = max(self._workspace_bytes(size) for size in {1, *sizes})
        self._room = [sizes[0], sizes[0] if len(sizes) > 1 else 1][: self.copies]
        self._stores = [None] * self.copies      # allocated when a plan first uses them
        self._plans = {}
        self._main = self._plan(sizes[0])        # the plan of a whole step's phases
        # side streams: `side` for the per-example phase, `side_b` for the clipped-sum phase
        self.side = [torch.cuda.Stream(device=dev) for _ in range(self.n_streams)] if self.n_streams > 1 else []
        # (three clipped-sum streams for eight per-example streams: measured 3 % better over the whole step than four)
        self.side_b = [torch.cuda.Stream(device=dev) for _ in range(max(2, 3 * self.n_streams // 8))] if self.n_streams > 1 else []
        # optional fused optimiser step (enable_update): parameters and momentum buffer, laid out like acc
        self.theta = None
        self.velocity = None
        self._update = None                      # (lr, momentum, keep_gradient)
        self._addresses = None                   # (stream, example addresses) of a step that is issued call by call
        self._recorded_addresses = []            # and those of steps that a caller records in a graph of its own
        self._phases = 0                         # phases issued since begin_step
        self._sum_plan = None                    # plan of the last of them
        self._last_sqnorm = torch.zeros((self.n_groups, self.rows), dtype=f32, device=dev)
        self._group_sqnorm = [self._last_sqnorm] * self.copies      # of the last micro-steps (one per copy)
        self._last = 0                           # the most recent one
        self._g_last = None                      # the stored gradients among them, and the plan that they were stored by
        self._g_plan = None
        self._not_stored = None                  # phase and inputs of a last micro-step whose gradients are not all stored (within a step)
        self.graph = None
        self.micro_steps_done = 0
        # Optimiser-step counter: the `step` word of the Philox counters.  The kernels read it from a device
        # word, so a captured graph draws fresh noise on every replay; finalize() advances it, `step` mirrors
        # it on the host.  Two optimiser steps never share a noise draw.
        self.step = int(wl.step)
        self._step_dev = torch.tensor([self.step], dtype=torch.int64, device=dev)
        # optional timing probe (bench.py): an object with arm(variant, flops, bytes) that asks the
        # library to bracket the next contraction kernel with a pair of events
        self.probe = None

    def _work(self, tensors: int, more: bool = False):
        """Algorithmic work of one call per layer: (flop, HBM bytes of the per-example call, HBM bytes of the
        recomputing clipped-sum call).  Bytes = the operands read once, plus the per-example gradients
        written when the layer materialises them, or the accumulator read and written by the recomputing form."""
        n, esize = self.wl.n * tensors, 2 if self.wl.dtype == "bf16" else 4
        return [(l.flops * n,
                 l.in_bytes(esize) * n + (4 * n * (pw + pb) if form == "materialise" else 0),
                 l.in_bytes(esize) * n + 8 * (pw + pb))
                for l, pw, pb, form in zip(self.layers, self.pw, self.pb, self._forms(tensors, more))]

    def _forms(self, tensors: int, more: bool = False) -> List[str]:
        """Form of every layer's clipped sum in a phase of `tensors` micro-steps: that of a micro-step, except that a phase of many
        one- or two-example micro-steps (which store every gradient) recomputes what a micro-step of that many examples would, where
        finished fp32 blocks are squared and scaled (how many micro-steps share a phase must not decide about precision) and the workspaces
        fit where the gradients would have been.  Stored, a layer's gradients cross memory twice; ResNet-50, us per step on four streams, every
        gradient stored / this: 3 x 1 364 / 362, 4 x 1 425 / 395, 8 x 1 693 / 548, 64 x 1 4099 / 2467; 3 x 2 at 192 x 192 574 / 491.  Not two
        micro-steps, half of which _last_plan stores all the same: 2 x 2 on one stream 544 / 555, at 192 x 192 532 / 559."""
        n = self.wl.n * tensors
        more = more and self.wl.accum > 1            # (workspaces have room for it)
        if more and tensors not in self._lean_forms:
            # A phase that others follow keeps no gradients of the layers whose clipped sum the whole-row kernel makes from finished fp32 blocks (the
            # same precision): 8 bytes per value and example less through memory.  ResNet-50, us a step on eight streams, every phase stores / this:
            # 8 x 32 6680 / 6360, 2 x 48 2700 / 2660; with GroupNorm 2 x 24 1940 / 1905; 8 x 24 on one stream 5960 / 5840.  The last one stores: `g` is whole
            # after a step.
            form = self._forms(tensors)
            rows = [] if self._mode != "auto" or self.clip_unit > 1 or form is not self.form or any(p % 4 for p in self.pw + self.pb) else (
                self._in_whole_rows([B.dp_kernel_variant(B.make_desc(l, n, self.wl.dtype), B.DP_WS_RECOMPUTE | B.DP_VARIANT_SHARED) for l in self.layers], n))
            rows = [i for i in rows if form[i] == "materialise"]
            self._lean_forms[tensors] = ["recompute" if i in rows else f for i, f in enumerate(form)] if rows else form
        if more:
            return self._lean_forms[tensors]
        if (tensors < 3 or self._mode != "auto" or self.wl.n > 2 or self.clip_unit > 1 or
                any(p % 4 for p in self.pw + self.pb)):         # (zeros between tensors have a place of their own in the matrix)
            return self.form
        if tensors not in self._phase_forms:
            norms, sums = (use | B.DP_RECOMPUTE_BLOCKS for use in (B.DP_WS_PER_EXAMPLE_GRAD, B.DP_WS_RECOMPUTE))
            over = {}                            # layer -> workspace less its part of the matrix
            descs = [B.make_desc(l, n, self.wl.dtype) for l in self.layers]
            variants = [B.dp_kernel_variant(d, sums | B.DP_VARIANT_SHARED) for d in descs]
            rows = self._in_whole_rows(variants, n)
            for i, (l, d, variant) in enumerate(zip(self.layers, descs, variants)):
                if variant and (i in rows or self._choose(l, "auto", n) == "recompute"):
                    need = max(B.dp_batch_workspace_bytes(d, norms), B.dp_workspace_bytes(d, sums), 16)
                    over[i] = _align256(need) - 4 * n * (self.pw[i] + self.pb[i])
            while over and sum(over.values()) + 256 > 0:
                del over[max(over, key=over.get)]
            self._phase_forms[tensors] = ["recompute" if i in over else form for i, form in enumerate(self.form)] if over else self.form
        return self._phase_forms[tensors]

    def _in_whole_rows(self, variants: Sequence[str], n: int) -> List[int]:
        """Layers that run in the whole-row kernel when the recomputing calls of `n` examples hold all that could (at most 16 a call)."""
        ids = [i for i, v in enumerate(variants) if "128x256rows" in v and n >= 12]
        calls, least = [ids[k: k + 16] for k in range(0, len(ids), 16)], ROWS_WORK[0 if n >= 17 else 1] * 768 * 2 * 128 * 128 * 64
        return [i for call in calls if len(call) > 1 and n * sum(self.layers[i].flops for i in call) >= least for i in call]

    def _blocks(self, tensors: int) -> int:
        """Or-ed into the uses of a phase's calls: whether it works on finished blocks."""
        return B.DP_RECOMPUTE_BLOCKS if self._forms(tensors) is not self.form else 0

    def _in_matrix(self, tensors: int) -> List[bool]:
        """Layers whose workspace lies in the gradient matrix: those that do not use their columns of it in such a phase and need
        more than they would if they did."""
        if self._forms(tensors) is self.form:
            return [False] * len(self.layers)
        if tensors not in self._inside:
            descs, need = self._workspaces(tensors)
            self._inside[tensors] = [now != form and b > max(16, B.dp_batch_workspace_bytes(d, B.DP_WS_PER_EXAMPLE_GRAD | B.DP_RECOMPUTE_BLOCKS))
                                     for d, b, now, form in zip(descs, need, self._forms(tensors), self.form)]
        return self._inside[tensors]

    def _columns(self, form: Sequence[str]):
        """Offsets of the layers' tensors (weight, bias) when the materialised ones lie side by side, and how many columns they have."""
        off_w, off_b, pos = [0] * len(self.layers), [0] * len(self.layers), 0
        for i in sorted((i for i, f in enumerate(form) if f == "materialise"), key=lambda i: self.off_w[i]):
            off_w[i] = pos
            off_b[i] = pos + _pad4(self.pw[i])
            pos = off_b[i] + _pad4(self.pb[i])
        return off_w, off_b, pos

    def _segments(self, form: Sequence[str], off_w: Sequence[int]):
        """Runs of columns of the gradient matrix that belong to one clipping group and lie side by side in the accumulator."""
        mat = sorted((i for i, f in enumerate(form) if f == "materialise"), key=lambda i: off_w[i])
        runs = [i for k, i in enumerate(mat) if k == 0 or self.group_of_layer[i] != self.group_of_layer[mat[k - 1]] or
                off_w[i] - off_w[mat[k - 1]] != self.off_w[i] - self.off_w[mat[k - 1]]]
        groups = [self.group_of_layer[i] for i in runs]
        return B.SegmentTable([off_w[i] for i in runs], groups, [self.group_clip[k] for k in groups], [self.off_w[i] for i in runs])

    def _workspaces(self, tensors: int):
        """Descriptors and workspace bytes of every layer in a phase of `tensors` micro-steps (the same whether others follow)."""
        if tensors not in self._needs:
            descs = [B.make_desc(l, self.wl.n * tensors, self.wl.dtype) for l in self.layers]
            blocks = self._blocks(tensors)
            need = [max(16, B.dp_batch_workspace_bytes(d, B.DP_WS_PER_EXAMPLE_GRAD | blocks),
                        B.dp_workspace_bytes(d, B.DP_WS_RECOMPUTE | blocks) if form == "recompute" else 0,
                        B.dp_batch_workspace_bytes(d, B.DP_WS_PER_EXAMPLE_GRAD, self.clip_unit) if self.clip_unit > 1 else 0)
                    for d, form in zip(descs, self._forms(tensors, True))]
            self._needs[tensors] = descs, need
        return self._needs[tensors]

    def _workspace_bytes(self, tensors: int) -> int:
        if tensors not in self._ws_bytes:
            self._ws_bytes[tensors] = sum(_align256(b) for b, inside in zip(self._workspaces(tensors)[1], self._in_matrix(tensors)) if not inside)
        return self._ws_bytes[tensors]

    def _micro_steps_together(self) -> int:
        """Micro-steps per phase, at most."""
        wl = self.wl
        if sum(self._example_bytes) * wl.n > PHASE_MICRO_STEP_BYTES:
            return 1
        most = max(1, (PHASE_EXAMPLES_OF_SMALL if wl.n <= 2 else PHASE_EXAMPLES) // wl.n)
        matrix = 4 * self.rows * self.p_mat
        phases = max(1, -(-wl.accum // most))
        alone = None
        while True:
            size = max(1, -(-wl.accum // phases))
            if size == 1:
                return 1
            copies = self.copies if phases > 1 else 1
            if copies * (size * matrix + self._workspace_bytes(size)) <= PHASE_STORE_BYTES:
                if alone is None:
                    alone = self._gathers(1)
                if not any(now and not before for now, before in zip(self._gathers(size), alone)):
                    return size
            phases += 1

    def _gathers(self, tensors: int) -> List[bool]:
        """Which calls of a phase of `tensors` micro-steps run the gathering kernel for want of room for rewritten operands (bf16 only): per
        layer the per-example and the recomputing one."""
        flags = []
        if self.wl.dtype == "bf16":
            blocks = self._blocks(tensors)
            for d, form in zip(self._workspaces(tensors)[0], self._forms(tensors)):
                stored = B.DP_VARIANT_MATERIALISE if form == "materialise" else 0
                flags.append("gather" in B.dp_kernel_variant(d, B.DP_WS_PER_EXAMPLE_GRAD | blocks | B.DP_VARIANT_SHARED | stored))
                flags.append(form == "recompute" and "gather" in B.dp_kernel_variant(d, B.DP_WS_RECOMPUTE | blocks | B.DP_VARIANT_SHARED))
        return flags

    def _phase_sizes(self, micro_steps: int) -> List[int]:
        """How many micro-steps each phase of a step of `micro_steps` holds: as few phases as the bounds allow, of nearly equal
        size."""
        phases = max(1, -(-micro_steps // self._together))
        while True:
            sizes = [micro_steps // phases + (1 if k < micro_steps % phases else 0) for k in range(phases)]
            # (the workspaces of a smaller phase may need more than those of the sizes that the buffers were made for)
            if self._ws_room is None or sizes[0] <= 1 or all(self._workspace_bytes(size) <= self._ws_room for size in set(sizes)):
                return sizes
            phases += 1

    def _plan(self, tensors: int, more: bool = False) -> _Plan:
        """Of phases of `tensors` micro-steps; more: of those that others of their step follow."""
        key = (tensors, more)
        if key not in self._plans and more and self._forms(tensors, True) is self._forms(tensors):
            self._plans[key] = self._plan(tensors)
        if key not in self._plans:
            stores = []
            for c, room in enumerate(self._room):
                if tensors <= room:
                    if self._stores[c] is None:
                        ws = self._workspace_bytes(1) if room == 1 else self._ws_room
                        self._stores[c] = _Store(self, room * self.rows, ws)
                    stores.append(self._stores[c])
            self._plans[key] = _Plan(self, tensors, stores, None, more)
        return self._plans[key]

    def _last_plan(self, form: Sequence[str]) -> _Plan:
        """Stores the gradients of one micro-step's layers that a phase of this form recomputes: whoever looks at `g` after a step finds the last
        micro-step's whole, as a micro-step of one or two examples leaves it.  Buffers of its own (one matrix of a micro-step beside those of
        the phase), so that its calls run beside the clipped sum: on the main stream, which has nothing else to do then (ResNet-50, 64 x 1 on four
        streams: 2454 us without them, 2467 so, 2735 on the streams of the per-example phase; 8 x 1 515, 548, 728)."""
        layers = tuple(i for i, f in enumerate(form) if f != self.form[i])
        if layers not in self._last_plans:
            if self._last_store is None:
                self._last_store = _Store(self, self.rows, self._workspace_bytes(1))
            self._last_plans[layers] = _Plan(self, 1, [self._last_store], layers)
        return self._last_plans[layers]

    # ---- one micro-step
    @property
    def descs(self):
        return self._workspaces(1)[0]

    @property
    def work(self):
        """Per layer: flop of one call, HBM bytes of the per-example call, HBM bytes of the recomputing clipped-sum call."""
        return self._work(1)

    @property
    def _g(self):
        """The gradient matrices; a micro-step's rows are the first ones of a phase."""
        return [st.g if st is not None else None for st in self._stores]

    @property
    def micro_steps_per_phase(self):
        return self._main.tensors

    def _arm(self, plan: _Plan, group, use: int):
        if self.probe is not None and group["conv"]:
            self.probe.arm(group["name"], sum(plan.work[i][0] for i in group["layers"]),
                           sum(plan.work[i][1 + use] for i in group["layers"]), len(group["layers"]))

    def _choose(self, layer, mode: str, n: int) -> str:
        if mode in ("materialise", "recompute"):
            return mode
        if mode != "auto":
            raise ValueError(mode)
        # Cost model fitted to the measured throughput of whole replayed steps on MI355X (micro-batch n, layers launched
        # in groups, kernels of several streams overlapping):
        #   materialise: the [n, P] fp32 gradients are written by the contraction's epilogue and read back by the
        #     streaming accumulate -- 8 n P bytes at ~5 TB/s;
        #   recompute: a second (clip-weighted) contraction -- the layer's inputs once more at ~4 TB/s and its flops
        #     at ~275 TFLOP/s sustained (no fixed cost: the weighted kernels run one example range per tile inside
        #     batch calls, without partial blocks or slice sums).
        # ResNet-50 at n = 32: the stride-1 3x3 layers of stage 3, stage 4 but its first 1x1 layer, and the classifier
        # recompute (15 layers, 19.4 M parameters).  Whole-step throughput around this split: 37/17 (300 TFLOP/s: the
        # strided 3x3 layer of stage 3, whose weighted form has no raw-row kernel, and the first 1x1 of stage 4 recompute
        # too) - 2 %, 44/10 (250) - 9 %, 26/28 (360) - 3 %.
        if n <= 2:
            # micro-steps of one or two examples are bound by their launches, and a recomputing layer brings launches of its
            # own to the clipped-sum phase (measured: 5.9 k against 5.6 k examples/s with the split above)
            return "materialise"
        p = layer.pw + layer.pb
        esize = 2 if self.wl.dtype == "bf16" else 4
        materialise = 8.0 * p * n / 5.0e12
        recompute = layer.in_bytes(esize) * n / 4.0e12 + layer.flops * n / 275.0e12
        return "materialise" if materialise <= recompute else "recompute"

    # ---- views of one layer's tensors in the flat vectors
    def acc_w(self, li: int) -> torch.Tensor:
        return self.acc[self.off_w[li]: self.off_w[li] + self.pw[li]]

    def acc_b(self, li: int) -> Optional[torch.Tensor]:
        return self.acc[self.off_b[li]: self.off_b[li] + self.pb[li]] if self.pb[li] else None

    def out_w(self, li: int) -> torch.Tensor:
        return self.out[self.off_w[li]: self.off_w[li] + self.pw[li]]

    def out_b(self, li: int) -> Optional[torch.Tensor]:
        return self.out[self.off_b[li]: self.off_b[li] + self.pb[li]] if self.pb[li] else None

    @property
    def group_sqnorm(self) -> torch.Tensor:
        """[groups, n] squared norms of the most recent micro-step."""
        return self._group_sqnorm[self._last]

    @property
    def g(self) -> Optional[torch.Tensor]:
        """[rows, p_mat] stored gradients of the most recent micro-step, columns as in the accumulator."""
        plan = self._g_plan
        if self._g_last is None or plan.form is self.form:
            return self._g_last
        # the phase stored some of the columns side by side, the others lie in a matrix of their own already
        out = self._last_store.g
        if plan.p_mat:
            for at, to, end in zip(plan.segments.begin, plan.segments.place, [*plan.segments.begin[1:], plan.p_mat]):
                out[:, to: to + end - at] = self._g_last[:, at: end]
        return out

    def enable_update(self, lr: float, momentum: float = 0.0, theta: Optional[torch.Tensor] = None,
                      keep_gradient: bool = True):
        """Make finalize() apply the SGD step in the same kernel (dp_add_noise_finalize_update): theta and the
        momentum buffer are flat vectors laid out like the accumulator.  `lr` can be changed per step with set_lr."""
        self.theta = torch.zeros_like(self.acc) if theta is None else theta
        self.velocity = torch.zeros_like(self.acc) if momentum != 0.0 else None
        self._update = [float(lr), float(momentum), bool(keep_gradient)]

    def set_lr(self, lr: float):
        self._update[0] = float(lr)

    def theta_w(self, li: int) -> torch.Tensor:
        return self.theta[self.off_w[li]: self.off_w[li] + self.pw[li]]

    def theta_b(self, li: int) -> Optional[torch.Tensor]:
        return self.theta[self.off_b[li]: self.off_b[li] + self.pb[li]] if self.pb[li] else None

    def set_step(self, step: int):
        """Set the optimiser-step counter (e.g. when a run is resumed)."""
        self.step = int(step)
        self._step_dev.fill_(self.step)

    def begin_step(self):
        self.acc.zero_()
        self.micro_steps_done = 0
        self._phases = 0
        self._sum_plan = None
        for store in self._stores:
            if store is not None:
                store.done = None

    def micro_step(self, inputs: Sequence):
        """inputs: per layer (x, dy) device tensors of the workload's dtype, n examples each.

        Phase A (per-example gradients + norms of every layer) and phase B (clipped sum) of one
        micro-step are separated by the norm reduction.  Layers within a phase are independent; with side
        streams they are spread over them, and phase A of the next micro-step does not wait for
        phase B of this one (they work on different buffer copies).  The clipped sums reach the
        accumulator in the same order on every run: each tensor is updated by one call per
        phase, issued on the same stream by every phase of one plan and behind all clipped sums of the phase before where the
        plan changes."""
        self._micro_step(inputs, False)

    def _micro_step(self, inputs: Sequence, more: bool):
        layers = range(len(self.layers))
        self._issue(self._plan(1, more), [inputs[i][0].data_ptr() for i in layers], [inputs[i][1].data_ptr() for i in layers], ends_step=not more)

    def _issue(self, plan: _Plan, x: Sequence[int], dy: Sequence[int], ends_step: bool = True):
        """The two phases of plan.tensors micro-steps; x, dy: per layer the address of the tensor, or of its array of example
        addresses.  ends_step: a caller may look at the last micro-step's norms afterwards."""
        at = plan.tensors > 1
        L = len(self.layers)
        gs = plan.p_mat
        c = self._phases % len(plan.stores)
        store = plan.stores[c]
        g_buf, gsq = plan.g[c], plan.group_sqnorm[c]
        fork = self.fork or ("step" if plan.n <= 2 else "micro_step")
        main = torch.cuda.current_stream()
        ms = main.cuda_stream
        # ---- phase A
        for st in self.side:
            if fork == "micro_step" or self._phases == 0:
                st.wait_stream(main)
            if store.done is not None:                # this copy's previous clipped sum has finished
                for ev in store.done:
                    st.wait_event(ev)
        # unit sums and their norms: one batch call per kernel variant, dealt to the side streams
        for grp in plan.groups_u:
            bt = grp["batch"][c]
            B.dp_unit_grad_batch(bt, self.clip_unit, bt.fill("x", [x[i] for i in grp["layers"]]), bt.fill("dy", [dy[i] for i in grp["layers"]]),
                                 grp["gw"][c], grp["gb"][c], grp["usq"][c], g_stride=gs,
                                 stream=self.side[grp["lane"]].cuda_stream if self.side else ms, addresses=at)
        for grp in plan.groups_a:
            bt = grp["batch"][c]
            self._arm(plan, grp, 0)
            B.dp_per_example_grad_batch(bt, bt.fill("x", [x[i] for i in grp["layers"]]), bt.fill("dy", [dy[i] for i in grp["layers"]]),
                                        grp["gw"][c], grp["gb"][c], None, g_stride=gs,
                                        stream=self.side[grp["lane"]].cuda_stream if self.side else ms, addresses=at)
            if not grp["counted"]:                     # how many partial sums per example each layer leaves behind
                for k, i in enumerate(grp["layers"]):
                    for table in plan.partials:
                        table.counts[i] = bt.partial_counts[k]
                grp["counted"] = True
        for st in self.side:
            main.wait_stream(st)
        # H2: every layer's partial sums -> per-group norms
        if self.clip_unit == 1:
            B.dp_norms_from_partials(plan.partials[c], plan.n, self.n_groups, gsq, stream=ms)
        else:
            B.dp_norms(plan.layer_sqnorm[c], self.group_of_layer_dev, L, plan.rows, self.n_groups, gsq, stream=ms)
        # ---- phase B
        sb = self.side_b
        if self._sum_plan not in (None, plan):
            # another plan deals the layers to other streams: what it still adds to a tensor comes first (by way of the main
            # stream, as everywhere else: in a captured step side streams must not wait for one another in a ring)
            self._drain()
        self._sum_plan = plan
        for st in sb:
            st.wait_stream(main)
        if gs:
            # one launch over all materialised tensors, whatever their clipping groups
            B.dp_clip_accumulate_columns(g_buf, gsq, self.n_groups, plan.segments, plan.rows, plan.rows // plan.tensors, gs, self.acc,
                                         g_stride=gs, stream=sb[0].cuda_stream if sb else ms)
        if self.noise == "per_example":
            for li in range(L):
                if plan.form[li] == "materialise":
                    self._example_noise(plan, li, sb[0].cuda_stream if sb else ms)
        for gi, grp in enumerate(plan.groups_b):
            st = sb[(1 + gi) % len(sb)].cuda_stream if sb else ms
            bt = grp["batch"][c]
            self._arm(plan, grp, 1)
            B.dp_clip_accumulate_recompute_batch(bt, bt.fill("x", [x[i] for i in grp["layers"]]), bt.fill("dy", [dy[i] for i in grp["layers"]]),
                                                 grp["sq"][c], grp["clip"], grp["acc_w"], grp["acc_b"], stream=st, addresses=at)
            if self.noise == "per_example":
                for li in grp["layers"]:
                    self._example_noise(plan, li, st)
        if sb:
            evs = []
            for st in sb:
                ev = torch.cuda.Event()
                ev.record(st)
                evs.append(ev)
            store.done = evs
        self._not_stored = (plan, x, dy) if plan.form is not self.form else None
        if ends_step:
            self._store_last()
        for k in range(max(0, plan.tensors - self.copies), plan.tensors):
            self._last = (self.micro_steps_done + k) % self.copies
            self._group_sqnorm[self._last] = gsq[:, k * self.rows:(k + 1) * self.rows]
        # the last micro-step's norms are a matrix of their own, as its callers read it
        if ends_step and not self._group_sqnorm[self._last].is_contiguous():
            self._last_sqnorm.copy_(self._group_sqnorm[self._last])
            self._group_sqnorm[self._last] = self._last_sqnorm
        self._g_last, self._g_plan = g_buf[-self.rows:] if g_buf is not None else None, plan
        self.micro_steps_done += plan.tensors
        self._phases += 1

    def _store_last(self):
        """The gradients of the last micro-step's layers that the last phase did not store."""
        if self._not_stored is None:
            return
        plan, x, dy = self._not_stored
        self._not_stored = None
        at = plan.tensors > 1
        skip = 8 * (plan.n - self.n) if at else 0      # entries of the tables before the last micro-step's examples
        for grp in self._last_plan(plan.form).groups_a:
            bt = grp["batch"][0]
            B.dp_per_example_grad_batch(bt, bt.fill("x", [x[i] + skip for i in grp["layers"]]), bt.fill("dy", [dy[i] + skip for i in grp["layers"]]),
                                        grp["gw"][0], grp["gb"][0], None, g_stride=self.p_mat, stream=torch.cuda.current_stream().cuda_stream, addresses=at)

    def _example_noise(self, plan: _Plan, li: int, st: int):
        """Per-example noise of this phase's examples for the tensors of layer li, on the stream that
        updates those tensors."""
        wl = self.wl
        first = self.micro_steps_done * self.n
        B.dp_add_example_noise(self.acc_w(li).data_ptr(), self.pw[li], wl.sigma, self.clip_total, wl.total_batch,
                               wl.philox_seed, 0, 2 * li, first, plan.n, step_dev=self._step_dev, stream=st)
        if self.pb[li]:
            B.dp_add_example_noise(self.acc_b(li).data_ptr(), self.pb[li], wl.sigma, self.clip_total, wl.total_batch,
                                   wl.philox_seed, 0, 2 * li + 1, first, plan.n, step_dev=self._step_dev, stream=st)

    def _drain(self):
        """The current stream waits for every clipped sum issued so far."""
        main = torch.cuda.current_stream()
        for st in self.side_b:
            main.wait_stream(st)

    def finalize(self):
        """H5 on the whole flat parameter vector in one launch (every tensor keeps its own Philox counters),
        with the SGD step fused in when enable_update() was called; then the step counter advances."""
        wl = self.wl
        self._drain()
        sigma = wl.sigma if self.noise == "once" else 0.0        # per-example form: the noise is already in acc
        if self._update is None:
            B.dp_add_noise_finalize_flat(self.acc, self.out, self._tensors, sigma, self.clip_total, wl.total_batch,
                                         wl.philox_seed, step_dev=self._step_dev)
        else:
            lr, momentum, keep = self._update
            B.dp_add_noise_finalize_flat(self.acc, self.out if keep else None, self._tensors, sigma, self.clip_total,
                                         wl.total_batch, wl.philox_seed, step_dev=self._step_dev, theta=self.theta,
                                         velocity=self.velocity, lr=lr, momentum=momentum)
        self._step_dev.add_(1)
        self.step += 1

    def _write_addresses(self, steps: Sequence[Sequence], sizes: List[int], table: torch.Tensor) -> torch.Tensor:
        """Example addresses of every operand (x and dy of each layer) of every phase: [operand][example of the phase], phase after
        phase."""
        operands, n = 2 * len(self.layers), self.wl.n
        first = 0
        for size in sizes:
            part = steps[first: first + size]
            B.dp_example_addresses([inputs[i][k].data_ptr() for i in range(len(self.layers)) for k in (0, 1) for inputs in part],
                                   self._example_bytes, operands, size, n, table.data_ptr() + 8 * operands * n * first)
            first += size
        return table

    def _address_table(self, micro_steps: int) -> torch.Tensor:
        """Room for the example addresses of a step."""
        need = 2 * len(self.layers) * self.wl.n * micro_steps
        if torch.cuda.is_current_stream_capturing():
            # the recorded launches write and read this table on every replay of a graph that is not ours: it stays
            table = torch.empty(need, dtype=torch.int64, device=self.device)
            self._recorded_addresses.append(table)
            return table
        # used again by the next step: whoever reads it has been waited for on this stream (finalize)
        stream = torch.cuda.current_stream().cuda_stream
        if self._addresses is None or self._addresses[0] != stream or self._addresses[1].numel() < need:
            self._addresses = stream, torch.empty(need, dtype=torch.int64, device=self.device)
        return self._addresses[1]

    def _issue_step(self, steps: Sequence[Sequence], table: Optional[torch.Tensor] = None):
        """Every micro-step of a step, several at a time where they are small (`table`: addresses already written).  A step that is broken off
        leaves the gradients of its last micro-step behind whole."""
        try:
            self._issue_phases(steps, table)
        finally:
            self._store_last()

    def _issue_phases(self, steps: Sequence[Sequence], table: Optional[torch.Tensor]):
        sizes = self._phase_sizes(len(steps))
        if max(sizes) <= 1:
            for k, inputs in enumerate(steps):
                self._micro_step(inputs, k + 1 < len(steps))
            return
        if table is None:
            table = self._write_addresses(steps, sizes, self._address_table(len(steps)))
        first, n, L = 0, self.wl.n, len(self.layers)
        for size in sizes:
            more = first + size < len(steps)
            if size == 1:
                self._micro_step(steps[first], more)
            else:
                base, row = table.data_ptr() + 8 * 2 * L * n * first, 8 * n * size
                self._issue(self._plan(size, more), [base + row * 2 * i for i in range(L)], [base + row * (2 * i + 1) for i in range(L)],
                            ends_step=not more)
            first += size

    def run(self, inputs_per_micro_step: Iterable[Sequence]):
        """One optimiser step.  A list or tuple holds the inputs of all micro-steps, which may then be issued together; from anything
        else they are taken, and issued, one by one (whoever makes them may use the same tensors again for the next)."""
        self.begin_step()
        if isinstance(inputs_per_micro_step, (list, tuple)):
            self._issue_step(inputs_per_micro_step)
        else:
            for inputs in inputs_per_micro_step:
                self.micro_step(inputs)
        self.finalize()
        return self.out

    def capture(self, inputs_per_micro_step: Iterable[Sequence]):
        """Record one whole optimiser step on these (persistent) input tensors into a HIP graph:
        replay() then re-issues every launch without host work.  Only kernels are recorded (the
        accumulator is cleared by a fill kernel, never by a memset node)."""
        assert self.probe is None or not getattr(self.probe, "enabled", False)
        step0 = self.step
        inputs_per_micro_step = list(inputs_per_micro_step)
        self.run(inputs_per_micro_step)          # warm-up outside capture (lazy module loads)
        sizes = self._phase_sizes(len(inputs_per_micro_step))
        table = None
        if max(sizes) > 1:
            need = 2 * len(self.layers) * self.wl.n * len(inputs_per_micro_step)
            table = self._write_addresses(inputs_per_micro_step, sizes, torch.empty(need, dtype=torch.int64, device=self.device))
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            self.begin_step()
            self._issue_step(inputs_per_micro_step, table)
            self.finalize()
        graph.example_addresses = table          # read by the recorded launches: kept as long as the graph is
        self.graph = graph
        self.set_step(step0)                     # recording consumed no optimiser step
        return graph

    def replay(self):
        """Re-issue the recorded step.  The step counter lives in device memory and is advanced by the graph
        itself, so every replay draws fresh noise."""
        self.graph.replay()
        self.step += 1
        return self.out

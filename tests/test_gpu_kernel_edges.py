"""GPU kernels at the edges of their tiles and of the rules that choose between them, against the oracle.

Tolerances: F32_TOL covers fp32 sums of up to a few thousand terms in any order (sqrt(K) 2^-24), BF16_TOL the one extra
rounding of scaled operands to bf16 (2^-9 per element)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2109_12191_amd as dp
from gpu_util import BF16_TOL, F32_TOL, assert_close, dev, host, launches
from test_gpu_kernels import _inputs, _oracle_grads, _run_per_example
from workloads import Layer, conv, dense, gn_affine, to_bf16_grid

pytestmark = pytest.mark.gpu


# vector widths 1, 2, 4, 8; teams from one lane to a wave; one, two and four waves per group; a last workgroup that is not full
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("c,hw,groups,n", [(6, 1, 3, 1), (6, 2, 3, 3), (4, 6, 2, 5), (65, 3, 1, 2), (129, 2, 1, 3), (256, 4, 1, 1),
                                           (64, 17, 32, 3), (2, 100, 1, 1), (9, 25, 3, 2), (512, 4, 32, 2)])
def test_groupnorm_lane_plans(c, hw, groups, n, dtype):
    tol = F32_TOL if dtype == "f32" else BF16_TOL
    layer = gn_affine(c, hw, groups)
    x, dy = _inputs(layer, n, 113, dtype)
    x = x * 1.5 + 0.25
    if dtype == "bf16":
        x = to_bf16_grid(x)
    ref_w, ref_b, ref_n2 = _oracle_grads(layer, x, dy)
    gw, gb, sq = _run_per_example(layer, x, dy, dtype)
    assert_close(gw, ref_w, tol, "dgamma")
    assert_close(gb, ref_b, tol, "dbeta")
    assert np.allclose(sq, ref_n2, rtol=tol)


# every team of 1 .. 64 lanes in a group that one wave has for itself (no barriers), and in one that the waves of a workgroup share
@pytest.mark.parametrize("cg,side", [(64, 1), (64, 2), (16, 2), (16, 3), (16, 8), (8, 5), (4, 7), (2, 11), (1, 13), (130, 2), (70, 3), (20, 5),
                                     (12, 7), (6, 11), (5, 13), (5, 16)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_groupnorm_teams(cg, side, dtype):
    layer = gn_affine(3 * cg, side, 3)
    x, dy = _inputs(layer, 3, 114, dtype)
    ref_w, ref_b, ref_n2 = _oracle_grads(layer, x, dy)
    gw, gb, sq = _run_per_example(layer, x, dy, dtype)
    tol = F32_TOL if dtype == "f32" else BF16_TOL
    assert_close(gw, ref_w, tol, "dgamma")
    assert_close(gb, ref_b, tol, "dbeta")
    assert np.allclose(sq, ref_n2, rtol=tol)


def _run_weighted(layer, x, dy, dtype, n2, clip_c):
    """acc_w, acc_b of the recomputing clipped sum, started from ones."""
    d = dp.make_desc(layer, x.shape[0], dtype)
    ws = torch.empty(max(16, dp.dp_workspace_bytes(d, dp.DP_WS_RECOMPUTE)), dtype=torch.uint8, device="cuda:0")
    acc_w = torch.ones(layer.pw, device="cuda:0")
    acc_b = torch.ones(max(4, layer.pb), device="cuda:0")
    dp.dp_clip_accumulate_recompute(d, dev(x, dtype), dev(dy, dtype), dev(n2.astype(np.float32)), clip_c, acc_w,
                                    acc_b if layer.pb else None, ws)
    torch.cuda.synchronize()
    assert torch.all(acc_b[layer.pb:] == 1.0)
    return host(acc_w), host(acc_b)[:layer.pb]


# tokens around the 16 of an MFMA step, the 32 / 64 of a staged step; features around the 64 of a tile and the four that a
# thread loads, odd and even rows; one example, fewer than the four groups of waves, more
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tokens,cin,cout,n", [(1, 64, 65, 1), (1, 130, 7, 37), (2, 3, 5, 3), (15, 66, 130, 4), (16, 64, 64, 5),
                                               (17, 101, 63, 3), (63, 65, 20, 2), (64, 128, 66, 6), (65, 33, 129, 7), (130, 70, 1, 9)])
def test_dense_token_kernels(tokens, cin, cout, n, dtype):
    layer = dense(cin, cout, tokens=tokens)
    x, dy = _inputs(layer, n, 117, dtype)
    ref_w, ref_b, ref_n2 = _oracle_grads(layer, x, dy)
    gw, gb, sq = _run_per_example(layer, x, dy, dtype)
    # bf16 products are exact in fp32: the fp32 bound holds for both input types
    assert_close(gw, ref_w, F32_TOL, "dW")
    assert_close(gb, ref_b, F32_TOL, "db")
    assert np.allclose(sq, ref_n2, rtol=F32_TOL)
    assert np.allclose(_run_per_example(layer, x, dy, dtype, materialise=False)[2], ref_n2, rtol=F32_TOL)
    clip_c = float(np.sqrt(np.median(ref_n2)))
    f = np.array([oracle.clip_factor(float(v), clip_c) for v in ref_n2])
    acc_w, acc_b = _run_weighted(layer, x, dy, dtype, ref_n2, clip_c)
    assert_close(acc_w, 1.0 + (f[:, None] * ref_w).sum(0), F32_TOL, "acc_w")
    assert_close(acc_b, 1.0 + (f[:, None] * ref_b).sum(0), F32_TOL, "acc_b")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tokens", [1, 3, 16, 70])
def test_dense_weighted_sum_leaves_out_an_example_that_overflows(tokens, dtype):
    """Finite inputs whose gradient does not fit fp32: the squared norm is infinite, the factor 0, and the sum is that of the others."""
    layer, n = dense(66, 70, tokens=tokens), 4
    x, dy = _inputs(layer, n, 119, dtype)
    ref_w, ref_b, ref_n2 = _oracle_grads(layer, x, dy)
    x[1], dy[1] = 2.0 ** 127, 2.0 ** 127
    n2 = ref_n2.copy()
    n2[1] = np.inf
    clip_c = float(np.sqrt(np.median(ref_n2)))
    f = np.array([oracle.clip_factor(float(v), clip_c) if np.isfinite(v) else 0.0 for v in n2])
    acc_w, acc_b = _run_weighted(layer, x, dy, dtype, n2, clip_c)
    assert_close(acc_w, 1.0 + (f[:, None] * ref_w).sum(0), F32_TOL, "acc_w")
    assert_close(acc_b, 1.0 + (f[:, None] * ref_b).sum(0), F32_TOL, "acc_b")


def test_packed_weighted_sum_keeps_the_neighbours_of_a_broken_example():
    """Operands packed into ranges of examples: an example whose norm is infinite or no number leaves the sum, its range does not."""
    layer, n = conv(64, 128, 3, 1, 13), 64
    name = dp.dp_kernel_variant(dp.make_desc(layer, n, "bf16"), dp.DP_WS_RECOMPUTE)
    assert name == "conv_contract<bf16,128x128,weighted>"
    x, dy = _inputs(layer, 8, 121, "bf16")
    ref_w, _, ref_n2 = _oracle_grads(layer, x, dy)
    x, dy, ref_w, n2 = (np.concatenate([v] * 8) for v in (x, dy, ref_w, ref_n2))
    n2[0], n2[3] = np.inf, np.nan
    clip_c = float(np.sqrt(np.median(ref_n2)))
    f = np.array([oracle.clip_factor(float(v), clip_c) if np.isfinite(v) else 0.0 for v in n2])
    acc_w, _ = _run_weighted(layer, x, dy, "bf16", n2, clip_c)
    assert_close(acc_w, 1.0 + (f[:, None] * ref_w).sum(0), BF16_TOL, "acc_w")


# ---- examples in several tensors (dp_example_addresses and the *_at calls): every kernel family, rows that start on odd
# elements, one example per tensor and several; the numbers are those of one tensor, bit for bit
def _addresses(tensors, n_per, example_bytes):
    table = torch.empty(len(tensors) * n_per, dtype=torch.int64, device="cuda:0")
    dp.dp_example_addresses([t.data_ptr() for t in tensors], [example_bytes], 1, len(tensors), n_per, table)
    assert table.tolist() == [t.data_ptr() + j * example_bytes for t in tensors for j in range(n_per)]
    return table


_SEVERAL = [
    ("1x1 64x64 tile", conv(64, 64, 1, 1, 12), "bf16"), ("1x1 128x128 odd tail", conv(160, 136, 1, 1, 10), "bf16"),
    ("1x1 256x128", conv(256, 256, 1, 1, 10), "bf16"), ("1x1 whole rows", conv(256, 512, 1, 1, 14), "bf16"),
    ("1x1 odd rows bias", conv(97, 71, 1, 1, 7, bias=True), "bf16"), ("1x1 stride 2", conv(48, 80, 1, 2, 14), "bf16"),
    ("1x1 stride 2 gram", conv(512, 256, 1, 2, 14), "bf16"), ("1x1 gram", conv(256, 512, 1, 1, 7), "bf16"),
    ("3x3 gram", conv(256, 512, 3, 1, 7), "bf16"), ("3x3 rows w7 odd channels", conv(65, 67, 3, 1, 7), "bf16"),
    ("3x3 rows w14", conv(64, 70, 3, 1, 14), "bf16"), ("3x3 rows w32 short", Layer("conv", 64, 64, 3, 32, 3, 3, 1, 1, False), "bf16"),
    ("3x3 rows s2", conv(64, 64, 3, 2, 28), "bf16"), ("3x3 general", conv(13, 70, 3, 1, 13), "bf16"),
    ("3x3 general s2 odd", conv(17, 33, 3, 2, 15, bias=True), "bf16"), ("5x5 stride 3", Layer("conv", 6, 10, 14, 17, 5, 5, 3, 2, True), "bf16"),
    ("tiny image", conv(3, 5, 3, 1, 3), "bf16"), ("stem", conv(3, 64, 7, 2, 64), "bf16"),
    ("fp32 3x3", conv(12, 20, 3, 1, 11, bias=True), "f32"), ("fp32 rows 3x3", conv(16, 16, 3, 1, 32), "f32"),
    ("fp32 rows 3x3 odd channels", conv(33, 15, 3, 1, 27, bias=True), "f32"), ("fp32 rows 5x5 s2", Layer("conv", 18, 20, 45, 37, 5, 5, 2, 2, True), "f32"),
    ("fp32 1x1", conv(70, 90, 1, 1, 8), "f32"),
    ("dense", dense(100, 37), "bf16"), ("dense fp32", dense(33, 70), "f32"), ("dense tokens odd", dense(37, 61, tokens=3), "bf16"),
    ("dense tokens", dense(66, 70, tokens=70), "bf16"), ("dense tokens fp32", dense(33, 30, tokens=5), "f32"),
    ("gn", gn_affine(32, 9, 8), "bf16"), ("gn fp32", gn_affine(16, 8, 4), "f32"), ("gn wide", gn_affine(600, 3, 2), "bf16"),
]


# maps of an odd number of values: channels start anywhere; one vector at each end, none between, several; a lane and a team per channel
@pytest.mark.parametrize("c,hw,groups,n", [(64, 7, 32, 3), (32, 13, 8, 2), (64, 5, 4, 5), (256, 25, 32, 1), (8, 14, 8, 3), (512, 6, 2, 2), (8, 45, 4, 2)])
def test_groupnorm_channels_that_start_anywhere(c, hw, groups, n):
    """bf16; what lies behind the inputs is not a number."""
    layer = gn_affine(c, hw, groups)
    x, dy = _inputs(layer, n, 117, "bf16")
    x = to_bf16_grid(x * 1.5 + 0.25)
    ref_w, ref_b, ref_n2 = _oracle_grads(layer, x, dy)
    own = [torch.full((a.size + 64,), float("nan"), dtype=torch.bfloat16, device="cuda:0") for a in (x, dy)]
    for t, a in zip(own, (x, dy)):
        t[: a.size] = dev(a, "bf16").view(-1)
    d = dp.make_desc(layer, n, "bf16")
    ws = torch.empty(max(16, dp.dp_workspace_bytes(d)), dtype=torch.uint8, device="cuda:0")
    g, sq = torch.zeros((n, 2 * c), device="cuda:0"), torch.zeros(n, device="cuda:0")
    dp.dp_per_example_grad(d, own[0], own[1], g, g[:, c:], sq, ws, g_stride=2 * c)
    torch.cuda.synchronize()
    assert_close(host(g[:, :c]), ref_w, F32_TOL, "dgamma")
    assert_close(host(g[:, c:]), ref_b, F32_TOL, "dbeta")
    assert np.allclose(host(sq), ref_n2, rtol=F32_TOL, atol=0)


@pytest.mark.parametrize("c,hw,groups,n", [(9, 7, 3, 9), (4, 5, 4, 11), (12, 13, 2, 5), (70, 9, 7, 3), (7, 6, 7, 7)])
def test_groupnorm_examples_whose_two_addresses_differ(c, hw, groups, n):
    """bf16 by address: X in a tensor per example, dY in one tensor whose examples start anywhere, and the other way round.  Waves of a
    workgroup have examples of both kinds."""
    layer = gn_affine(c, hw, groups)
    x, dy = _inputs(layer, n, 118, "bf16")
    x = to_bf16_grid(x * 1.5 + 0.25)
    ref_w, ref_b, ref_n2 = _oracle_grads(layer, x, dy)
    d = dp.make_desc(layer, n, "bf16")
    together = [dev(a, "bf16") for a in (x, dy)]
    each = [[t[i].clone() for i in range(n)] for t in together]
    tables = [[_addresses([t], n, 2 * t[0].numel()), _addresses(e, 1, 2 * t[0].numel())] for t, e in zip(together, each)]
    assert any((a ^ b) & 15 for a, b in zip(tables[0][0].tolist(), tables[0][1].tolist()))
    off_b = (c + 3) // 4 * 4
    width = 2 * off_b
    for kx, kd in ((0, 1), (1, 0), (0, 0)):
        need = dp.dp_workspace_bytes(d)
        ws = torch.empty(max(16, need), dtype=torch.uint8, device="cuda:0")
        g, sq = torch.full((n, width), 7.0, device="cuda:0"), torch.full((n,), -1.0, device="cuda:0")
        batch = dp.LayerBatch([d], [ws.data_ptr()], [ws.numel()])
        dp.dp_per_example_grad_batch(batch, batch.ptrs([tables[0][kx].data_ptr()]), batch.ptrs([tables[1][kd].data_ptr()]), batch.ptrs([g.data_ptr()]),
                                     batch.ptrs([g.data_ptr() + 4 * off_b]), batch.ptrs([sq.data_ptr()]), g_stride=width, addresses=True)
        torch.cuda.synchronize()
        assert_close(host(g[:, :c]), ref_w, F32_TOL, "dgamma")
        assert_close(host(g[:, off_b:off_b + c]), ref_b, F32_TOL, "dbeta")
        assert np.allclose(host(sq), ref_n2, rtol=F32_TOL, atol=0)


# Rows that are brought to another length: planes of whole pieces (1x1, 56- and 16-wide), of halves (28) and of neither (14, 7, parity
# split after it); fewer than 64 positions, one beyond a multiple of 8; strides with and without a remainder; the first convolution.
_WIDENED = [conv(64, 96, 1, 1, 7), conv(40, 33, 1, 1, 9), conv(33, 64, 1, 1, 13), conv(48, 80, 1, 2, 13), conv(32, 36, 1, 2, 26), conv(64, 64, 3, 1, 5),
            conv(64, 72, 3, 1, 13), conv(66, 64, 3, 1, 20), conv(64, 64, 3, 1, 15), conv(64, 64, 3, 1, 40), conv(64, 64, 3, 2, 13), conv(64, 65, 3, 2, 25),
            conv(64, 64, 3, 2, 40), Layer("conv", 64, 64, 9, 25, 3, 3, 1, 1, False), Layer("conv", 64, 64, 11, 12, 3, 3, 2, 1, False), conv(3, 64, 7, 2, 60)]


@pytest.mark.parametrize("several", [False, True])
@pytest.mark.parametrize("materialise", [False, True])
@pytest.mark.parametrize("room", [True, False])
def test_rows_brought_to_another_length(materialise, several, room):
    """In one batch call with room for the copies alone (F32_TOL: the products of bf16 inputs are exact, sums are fp32), examples in one
    tensor or each in one of its own.  What is around the inputs is not a number."""
    n = 13
    shared = dp.DP_WS_PER_EXAMPLE_GRAD | dp.DP_VARIANT_SHARED | (dp.DP_VARIANT_MATERIALISE if materialise else 0)
    descs = [dp.make_desc(l, n, "bf16") for l in _WIDENED]
    for l, d in zip(_WIDENED, descs):
        assert "gather" not in dp.dp_kernel_variant(d, shared), l
    ins = [_inputs(l, n, 30 + k, "bf16") for k, l in enumerate(_WIDENED)]
    kept, ptrs = [], [[], []]
    for pair in ins:
        for side, a in enumerate(pair):
            t, per = dev(a, "bf16").view(n, -1), a[0].size
            room = (per + 31) // 8 * 8
            if several:
                own = torch.full((n, 8 + room), float("nan"), dtype=torch.bfloat16, device="cuda:0")
                own[:, 8: 8 + per] = t
                table = torch.tensor([own[i, 8:].data_ptr() for i in range(n)], dtype=torch.int64, device="cuda:0")
                kept += [own, table]
                ptrs[side].append(table.data_ptr())
            else:
                own = torch.full((8 + n * per + 32,), float("nan"), dtype=torch.bfloat16, device="cuda:0")
                own[8: 8 + n * per] = t.reshape(-1)
                kept.append(own)
                ptrs[side].append(own[8:].data_ptr())
    sizes = [dp.dp_batch_workspace_bytes(d) if room else dp.dp_workspace_bytes(d) for d in descs]      # (without room: read in place)
    assert all(dp.dp_batch_workspace_bytes(d) > dp.dp_workspace_bytes(d) for d in descs)
    wss = [torch.full((b,), 255, dtype=torch.uint8, device="cuda:0") for b in sizes]
    stride = max(l.pw for l in _WIDENED) + 3 & ~3
    g = [torch.full((n, stride), float("nan"), dtype=torch.float32, device="cuda:0") for _ in descs]
    sq = torch.full((len(descs), n), -1.0, device="cuda:0")
    batch = dp.LayerBatch(descs, [w.data_ptr() for w in wss], sizes)
    dp.dp_per_example_grad_batch(batch, batch.ptrs(ptrs[0]), batch.ptrs(ptrs[1]), batch.ptrs([t.data_ptr() for t in g]) if materialise else None, None,
                                 batch.ptrs([sq[k].data_ptr() for k in range(len(descs))]), g_stride=stride if materialise else 0, addresses=several)
    torch.cuda.synchronize()
    for k, l in enumerate(_WIDENED):
        ref_w, _, ref_n2 = _oracle_grads(l, *ins[k])
        assert np.allclose(host(sq[k]), ref_n2, rtol=F32_TOL, atol=0), (k, l)
        if materialise:
            assert_close(host(g[k][:, : l.pw]), ref_w, F32_TOL, f"layer {k} {l}")


# Maps of 1, 9, 25, 49 and 64 positions in rows of 64; ragged channel counts below, at and beyond the tiles; strides with and without
# a remainder; aligned rows in place; dense layers of one and of several tokens.
_BLOCKS = [conv(128, 192, 1, 1, 7), conv(72, 136, 1, 2, 13), conv(80, 65, 1, 2, 9), conv(64, 96, 3, 1, 7), conv(40, 33, 3, 2, 14), conv(128, 64, 3, 1, 8),
           conv(64, 64, 3, 1, 3), conv(130, 60, 1, 1, 1), conv(48, 64, 1, 1, 10), dense(200, 70), dense(66, 130, 20)]


@pytest.mark.parametrize("layer", _BLOCKS, ids=str)
def test_clipped_sum_that_scales_finished_blocks(layer):
    """As exact as fp32 sums are: the products of bf16 inputs are exact, and each of the few additions per position and example
    rounds by 2^-24 of a partial sum (F32_TOL / 10, where operands scaled in bf16 would show 2^-9).  Layers share a launch with
    another one, examples lie in tensors of their own."""
    for n in (1, 5, 34):
        layers = [layer, _BLOCKS[0]]
        descs = [dp.make_desc(l, n, "bf16") for l in layers]
        use = dp.DP_WS_RECOMPUTE | dp.DP_RECOMPUTE_BLOCKS
        wss = [torch.empty(max(16, dp.dp_workspace_bytes(d, use)), dtype=torch.uint8, device="cuda:0").fill_(255) for d in descs]
        ins = [_inputs(l, n, 77 + k, "bf16") for k, l in enumerate(layers)]
        tensors = [[dev(a, "bf16").unbind(0) for a in pair] for pair in ins]
        tensors = [[[t.clone() for t in side] for side in pair] for pair in tensors]
        tables = [[torch.tensor([t.data_ptr() for t in side], dtype=torch.int64, device="cuda:0") for side in pair] for pair in tensors]
        n2 = (np.random.default_rng(7).uniform(0.4, 2.0, (2, n)) ** 2).astype(np.float32)
        n2[:, n // 2] = -1.0 if n > 1 else n2[:, 0]              # a broken example: factor 0
        n2d = dev(n2)
        acc_w = [torch.full((l.pw,), 0.125, dtype=torch.float32, device="cuda:0") for l in layers]
        acc_b = [torch.full((max(l.pb, 1),), 0.125, dtype=torch.float32, device="cuda:0") for l in layers]
        batch = dp.LayerBatch(descs, [w.data_ptr() for w in wss], [w.numel() for w in wss], scale_blocks=True)
        dp.dp_clip_accumulate_recompute_batch(batch, batch.ptrs([t[0].data_ptr() for t in tables]), batch.ptrs([t[1].data_ptr() for t in tables]),
                                              batch.ptrs([n2d[k].data_ptr() for k in range(2)]), batch.floats([1.0, 1.0]),
                                              batch.ptrs([t.data_ptr() for t in acc_w]),
                                              batch.ptrs([t.data_ptr() if l.pb else None for t, l in zip(acc_b, layers)]), addresses=True)
        torch.cuda.synchronize()
        for k, l in enumerate(layers):
            f = np.array([0.0 if v < 0 else oracle.clip_factor(float(v), 1.0) for v in n2[k]])
            ref_w, ref_b, _ = _oracle_grads(l, *ins[k])
            assert_close(host(acc_w[k]), 0.125 + (f[:, None] * ref_w).sum(axis=0), F32_TOL / 10, f"{l} n={n} weights")
            if l.pb:
                assert_close(host(acc_b[k])[:l.pb], 0.125 + (f[:, None] * ref_b).sum(axis=0), F32_TOL / 10, f"{l} n={n} bias")


@pytest.mark.parametrize("layer", [l for l in _BLOCKS if l.kind == "conv"], ids=str)
@pytest.mark.parametrize("kind", ["overflow", "infinite", "no number"])
def test_finished_blocks_of_a_broken_example_add_nothing(layer, kind):
    """Finite inputs whose gradient does not fit fp32, and inputs that are not finite: norm infinite or no number, factor 0, and the sum is that
    of the others."""
    n, bad = 6, 2
    x, dy = _inputs(layer, n, 123, "bf16")
    good = [i for i in range(n) if i != bad]
    ref_w = _oracle_grads(layer, x[good], dy[good])[0]
    x[bad], dy[bad] = 2.0 ** 127, 2.0 ** 127
    if kind != "overflow":
        x[bad, 0], dy[bad, -1] = np.inf if kind == "infinite" else np.nan, -np.inf
    n2 = (np.random.default_rng(9).uniform(0.4, 2.0, n) ** 2).astype(np.float32)
    n2[bad] = np.nan if kind == "no number" else np.inf
    d = dp.make_desc(layer, n, "bf16")
    ws = torch.empty(max(16, dp.dp_workspace_bytes(d, dp.DP_WS_RECOMPUTE | dp.DP_RECOMPUTE_BLOCKS)), dtype=torch.uint8, device="cuda:0")
    xd, dyd, n2d, acc = dev(x, "bf16"), dev(dy, "bf16"), dev(n2), torch.full((layer.pw,), 0.125, device="cuda:0")
    tables = [_addresses([t], n, 2 * t[0].numel()) for t in (xd, dyd)]
    batch = dp.LayerBatch([d], [ws.data_ptr()], [ws.numel()], scale_blocks=True)
    dp.dp_clip_accumulate_recompute_batch(batch, batch.ptrs([tables[0].data_ptr()]), batch.ptrs([tables[1].data_ptr()]), batch.ptrs([n2d.data_ptr()]),
                                          batch.floats([1.0]), batch.ptrs([acc.data_ptr()]), None, addresses=True)
    torch.cuda.synchronize()
    f = np.array([oracle.clip_factor(float(n2[i]), 1.0) for i in good])
    assert_close(host(acc), 0.125 + (f[:, None] * ref_w).sum(axis=0), F32_TOL / 10, "sum of the others")


# one value at a time (an odd number of columns); eight rows at a time and those that are left; several passes over the factors
@pytest.mark.parametrize("n,p", [(5, 7), (8, 64), (21, 4100), (1030, 12)])
def test_stored_clipped_sum_leaves_out_rows_that_are_not_finite(n, p):
    rng = np.random.default_rng(11)
    g, n2 = rng.standard_normal((n, p)).astype(np.float32), (rng.uniform(0.4, 2.0, n) ** 2).astype(np.float32)
    f = np.array([oracle.clip_factor(float(v), 1.0) for v in n2])
    for i, (value, norm) in {1: (np.inf, np.inf), 3: (np.nan, np.nan), n - 1: (-np.inf, -1.0)}.items():
        g[i, ::3], n2[i], f[i] = value, norm, 0.0
    want = 0.5 + (f[:, None] * np.where(f[:, None] > 0, g, 0.0)).sum(0)
    stride = (p + 3) // 4 * 4 if p > 7 else p
    gd = torch.zeros((n, stride), device="cuda:0")
    gd[:, :p] = dev(g)
    n2d, acc = dev(n2), torch.full((stride,), 0.5, device="cuda:0")
    dp.dp_clip_accumulate(gd, n2d, 1.0, n, p, acc, g_stride=stride)
    assert_close(host(acc[:p]), want, F32_TOL, "one group")
    if p % 4 == 0:
        acc.fill_(0.5)
        table = dp.SegmentTable([0, p // 8 * 4], [0, 0], [1.0, 1.0])
        dp.dp_clip_accumulate_segments(gd, n2d, 1, table, n, p, acc, g_stride=stride)
        assert_close(host(acc[:p]), want, F32_TOL, "segments")


def test_layers_that_cannot_scale_finished_blocks_are_refused():
    use = dp.DP_WS_RECOMPUTE | dp.DP_RECOMPUTE_BLOCKS
    for layer in (conv(64, 64, 3, 1, 14), conv(64, 64, 1, 1, 7, bias=True), conv(64, 64, 1, 1, 9)):
        d = dp.make_desc(layer, 4, "bf16")
        assert dp.dp_kernel_variant(d, use) == "" and dp.dp_workspace_bytes(d, use) == 0
        assert dp.dp_kernel_variant(dp.make_desc(layer, 4, "f32"), use) != ""
        t = torch.zeros(4, dtype=torch.int64, device="cuda:0")
        batch = dp.LayerBatch([d], [t.data_ptr()], [32], scale_blocks=True)
        acc = torch.zeros(layer.pw, dtype=torch.float32, device="cuda:0")
        with pytest.raises(dp.DpError):
            dp.dp_clip_accumulate_recompute_batch(batch, batch.ptrs([t.data_ptr()]), batch.ptrs([t.data_ptr()]), batch.ptrs([t.data_ptr()]),
                                                  batch.floats([1.0]), batch.ptrs([acc.data_ptr()]),
                                                  batch.ptrs([acc.data_ptr() if layer.pb else None]), addresses=True)


@pytest.mark.parametrize("n_per", [1, 3])
@pytest.mark.parametrize("name,layer,dtype", _SEVERAL, ids=[c[0] for c in _SEVERAL])
def test_examples_in_several_tensors(name, layer, dtype, n_per):
    tensors = 33 if name in ("1x1 256x128", "1x1 whole rows") else 120 if name.startswith("fp32 rows") else 4      # (those kernels want many tiles)
    n = tensors * n_per
    if name.startswith("fp32 rows"):
        assert dp.dp_kernel_variant(dp.make_desc(layer, n, dtype), dp.DP_WS_PER_EXAMPLE_GRAD).startswith("conv_rows<f32")
    x, dy = _inputs(layer, n, 131, dtype)
    xd, dyd = dev(x, dtype), dev(dy, dtype)
    es = 2 if dtype == "bf16" else 4
    x_parts = [xd[k * n_per:(k + 1) * n_per].clone() for k in range(tensors)]
    dy_parts = [dyd[k * n_per:(k + 1) * n_per].clone() for k in range(tensors)]
    xt, dyt = _addresses(x_parts, n_per, layer.x_bytes(es)), _addresses(dy_parts, n_per, layer.dy_bytes(es))
    d = dp.make_desc(layer, n, dtype)
    ws = torch.empty(max(16, dp.dp_workspace_bytes(d), dp.dp_workspace_bytes(d, dp.DP_WS_RECOMPUTE), dp.dp_unit_workspace_bytes(d, 3)),
                     dtype=torch.uint8, device="cuda:0")
    batch = dp.LayerBatch([d], [ws.data_ptr()], [ws.numel()])
    row = (layer.pw + 3) // 4 * 4
    got = []
    for addresses, xp, dyp in ((False, xd, dyd), (True, xt, dyt)):
        res = []
        g = torch.zeros((n, row + (layer.pb + 3) // 4 * 4), device="cuda:0")
        sq, sq2 = torch.zeros(n, device="cuda:0"), torch.zeros(n, device="cuda:0")
        args = (batch.ptrs([xp.data_ptr()]), batch.ptrs([dyp.data_ptr()]))
        gb = batch.ptrs([g[:, row:].data_ptr()]) if layer.pb else None
        dp.dp_per_example_grad_batch(batch, *args, batch.ptrs([g.data_ptr()]), gb, batch.ptrs([sq.data_ptr()]), g_stride=g.shape[1],
                                     addresses=addresses)
        dp.dp_per_example_grad_batch(batch, *args, None, None, batch.ptrs([sq2.data_ptr()]), addresses=addresses)
        acc, acc_b = torch.ones(row, device="cuda:0"), torch.ones(max(4, layer.pb), device="cuda:0")
        clip = float(sq.median().sqrt())
        dp.dp_clip_accumulate_recompute_batch(batch, *args, batch.ptrs([sq.data_ptr()]), batch.floats([clip]), batch.ptrs([acc.data_ptr()]),
                                              batch.ptrs([acc_b.data_ptr()]) if layer.pb else None, addresses=addresses)
        res = [g, sq, sq2, acc, acc_b]
        if n_per == 3:
            gu, squ = torch.zeros((tensors, g.shape[1]), device="cuda:0"), torch.zeros(tensors, device="cuda:0")
            dp.dp_unit_grad_batch(batch, 3, *args, batch.ptrs([gu.data_ptr()]), batch.ptrs([gu[:, row:].data_ptr()]) if layer.pb else None,
                                  batch.ptrs([squ.data_ptr()]), g_stride=g.shape[1], addresses=addresses)
            res += [gu, squ]
        torch.cuda.synchronize()
        got.append(res)
    for k, (one, several) in enumerate(zip(*got)):
        assert torch.isfinite(one).all() and torch.equal(one, several), k
    # and they are the right numbers (the other tests check the one-tensor calls; this guards against both reading nothing)
    if layer.pw * n < 4e6:
        ref_w, _, ref_n2 = _oracle_grads(layer, x[:2], dy[:2])
        assert_close(host(got[1][0])[:2, :layer.pw], ref_w, BF16_TOL, "dW")
        assert np.allclose(host(got[1][1])[:2], ref_n2, rtol=BF16_TOL)


def test_segments_at_places_of_their_own():
    """dp_clip_accumulate_columns: segments around the 1024 columns of a workgroup, moved in the accumulator, against numpy."""
    rng = np.random.default_rng(7)
    begins, groups, clips = [0, 4, 1028, 2052, 3080], [0, 2, 1, 0, 2], [1.0, 0.5, 2.0, 0.7, float("inf")]
    p, n = 4200, 18
    places = [8000, 4096, 0, 2048, 5800]
    g = rng.standard_normal((n, p + 4)).astype(np.float32)
    sq = rng.uniform(0.2, 3.0, (3, n)).astype(np.float32)
    acc0 = rng.standard_normal(8192).astype(np.float32)
    want = acc0.astype(np.float64)
    for k, b in enumerate(begins):
        e = (begins + [p])[k + 1]
        f = np.array([oracle.clip_factor(float(v), clips[k]) for v in sq[groups[k]]])
        want[places[k]: places[k] + e - b] += (f[:, None] * g[:, b:e].astype(np.float64)).sum(0)
    table, gd, sqd = dp.SegmentTable(begins, groups, clips, places), dev(g), dev(sq)
    for run in (1, 3, 9, 18):
        acc = dev(acc0)
        dp.dp_clip_accumulate_columns(gd, sqd, 3, table, n, run, p, acc, g_stride=p + 4)
        assert_close(host(acc), want, F32_TOL, "acc")
        split = dev(acc0)                              # the same runs, a call each: the same bits
        for k in range(0, n, run):
            dp.dp_clip_accumulate_columns(gd[k:], sqd[:, k:k + run].contiguous(), 3, table, run, run, p, split, g_stride=p + 4)
        assert torch.equal(acc, split), run


# ---- fp32 convolutions from raw rows: channels around the 16 and 32 of a block, output rows that are no multiple of four, one column,
# a kernel larger than the image, several chunks of rows with a short last one, several examples per workgroup (as many examples as
# the kernel is chosen for)
@pytest.mark.parametrize("cin,cout,h,w,k,stride,n", [(16, 16, 5, 7, 3, 2, 500), (33, 15, 8, 9, 3, 1, 200), (3, 16, 9, 6, 3, 1, 2000), (17, 13, 2, 1, 3, 1, 800),
                                                     (32, 32, 57, 56, 3, 1, 260), (48, 16, 33, 36, 3, 1, 50), (16, 48, 17, 13, 5, 2, 100),
                                                     (20, 31, 24, 26, 5, 1, 100), (5, 16, 46, 43, 5, 1, 100), (18, 20, 45, 37, 5, 2, 100),
                                                     (16, 16, 12, 14, 3, 1, 8200), (2, 3, 130, 260, 3, 1, 200)])
def test_conv_f32_raw_rows_kernel(cin, cout, h, w, k, stride, n):
    layer = Layer("conv", cin, cout, h, w, k, k, stride, (k - 1) // 2, cout % 2 == 0)
    assert dp.dp_kernel_variant(dp.make_desc(layer, n, "f32"), dp.DP_WS_PER_EXAMPLE_GRAD).startswith("conv_rows<f32")
    x, dy = _inputs(layer, min(n, 5), 131, "f32")
    if n > 5:                                     # the oracle's few examples, over and over
        x, dy = (np.concatenate([v] * (n // 5)) for v in (x, dy))
    gw, gb, sq = _run_per_example(layer, x, dy, "f32")
    norms = _run_per_example(layer, x, dy, "f32", materialise=False)[2]
    ref_w, ref_b, ref_n2 = _oracle_grads(layer, x[:5], dy[:5])
    for got, ref in ((gw, ref_w), (gb, ref_b), (sq, ref_n2)):
        if ref is not None and ref.size:
            got = got.reshape((-1,) + ref.shape)
            assert np.array_equal(got, np.broadcast_to(got[0], got.shape))      # the same bits wherever an example lies
            assert_close(got[0], ref, F32_TOL, "gradient")
    assert np.allclose(norms, sq, rtol=F32_TOL)


def test_conv_f32_raw_rows_kernel_in_a_batch_call():
    """Layers of every kernel size and stride in one batch call, where the kernel is planned for a chip that other layers fill."""
    n, few = 200, 5
    layers = [Layer("conv", ci, co, h, w, k, k, s, (k - 1) // 2, co % 2 == 0) for ci, co, h, w, k, s in
              [(33, 15, 8, 9, 3, 1), (48, 16, 33, 36, 3, 1), (16, 48, 17, 13, 5, 2), (20, 31, 24, 26, 5, 1), (5, 16, 46, 43, 5, 1), (18, 20, 45, 37, 5, 2),
               (16, 32, 32, 32, 3, 2), (40, 16, 13, 17, 3, 2)]]
    descs = [dp.make_desc(l, n, "f32") for l in layers]
    assert all(dp.dp_kernel_variant(d, dp.DP_WS_PER_EXAMPLE_GRAD | dp.DP_VARIANT_SHARED).startswith("conv_rows<f32") for d in descs)
    ins = [_inputs(l, few, 151 + k, "f32") for k, l in enumerate(layers)]
    xs, dys = ([dev(v[j]).repeat((n // few,) + (1,) * (v[j].ndim - 1)).contiguous() for v in ins] for j in (0, 1))
    ws = [torch.empty(max(16, dp.dp_workspace_bytes(d)), dtype=torch.uint8, device="cuda:0") for d in descs]
    batch = dp.LayerBatch(descs, [t.data_ptr() for t in ws], [t.numel() for t in ws])
    rows = [(l.pw + 3) // 4 * 4 for l in layers]
    pitch = max(r + (l.pb + 3) // 4 * 4 for r, l in zip(rows, layers))
    g = [torch.full((n, pitch), 7.0, device="cuda:0") for _ in layers]
    sq, norms = (torch.full((len(layers), n), -1.0, device="cuda:0") for _ in range(2))
    args = batch.ptrs([t.data_ptr() for t in xs]), batch.ptrs([t.data_ptr() for t in dys])
    dp.dp_per_example_grad_batch(batch, *args, batch.ptrs([t.data_ptr() for t in g]),
                                 batch.ptrs([t[:, r:].data_ptr() if l.pb else None for t, r, l in zip(g, rows, layers)]),
                                 batch.ptrs([sq[k].data_ptr() for k in range(len(layers))]), g_stride=pitch)
    dp.dp_per_example_grad_batch(batch, *args, None, None, batch.ptrs([norms[k].data_ptr() for k in range(len(layers))]))
    torch.cuda.synchronize()
    for k, (l, (x, dy)) in enumerate(zip(layers, ins)):
        ref_w, ref_b, ref_n2 = _oracle_grads(l, x, dy)
        assert torch.equal(g[k], g[k][:few].repeat(n // few, 1)) and torch.equal(sq[k], sq[k][:few].repeat(n // few))
        got = host(g[k][:few])
        assert_close(got[:, :l.pw], ref_w, F32_TOL, f"layer {k} dW")
        if l.pb:
            assert_close(got[:, rows[k]:rows[k] + l.pb], ref_b, F32_TOL, f"layer {k} db")
        assert np.allclose(host(sq[k][:few]), ref_n2, rtol=F32_TOL) and np.allclose(host(norms[k]), host(sq[k]), rtol=F32_TOL)


def test_conv_f32_raw_rows_kernel_keeps_what_is_not_finite_in_its_place():
    """An infinity in the last column of a row reaches the taps that read it and no other."""
    layer = Layer("conv", 32, 16, 3, 5, 3, 3, 1, 1, False)
    x, dy = _inputs(layer, 400, 137, "f32")
    assert dp.dp_kernel_variant(dp.make_desc(layer, 400, "f32"), dp.DP_WS_PER_EXAMPLE_GRAD).startswith("conv_rows<f32")
    dy[:] = 1.0
    x[0, 0, 1, 4] = np.inf
    gw = _run_per_example(layer, x, dy, "f32")[0].reshape(400, 16, 32, 3, 3)[0]
    want = np.ones((3, 3), bool)                  # the middle row, the last column: kw = 0 needs column 5 of dY, which is not there
    want[:, 0] = False
    assert np.array_equal(np.isinf(gw[0, 0]), want) and np.isfinite(gw[:, 1]).all() and np.isfinite(gw[:, 0, :, 0]).all()


# The products of the raw-row kernel run on parts of the numbers.  What they leave out is below 2^-23 of a product, and sums of 32 products are
# rounded into one fp32 sum of K / 32 (and 2 to 12 shares of it) terms: sqrt(K / 32) * 2^-24 at most, taken twice
@pytest.mark.parametrize("cin,cout,h,w,k,stride,n", [(64, 64, 56, 56, 3, 1, 100), (16, 16, 32, 32, 3, 1, 300), (17, 33, 30, 29, 3, 1, 300),
                                                     (40, 72, 45, 37, 5, 2, 40), (64, 32, 33, 34, 3, 2, 300), (20, 40, 28, 27, 5, 1, 100), (18, 20, 40, 3, 3, 1, 300)])
def test_conv_f32_raw_rows_kernel_is_as_exact_as_fp32(cin, cout, h, w, k, stride, n):
    layer = Layer("conv", cin, cout, h, w, k, k, stride, (k - 1) // 2, cout % 2 == 0)
    x, dy = (np.concatenate([v] * (n // 2)) for v in _inputs(layer, 2, 139, "f32"))
    assert dp.dp_kernel_variant(dp.make_desc(layer, n, "f32"), dp.DP_WS_PER_EXAMPLE_GRAD).startswith("conv_rows<f32")
    gw, gb, sq = _run_per_example(layer, x, dy, "f32")
    ref_w, ref_b, ref_n2 = _oracle_grads(layer, x[:2], dy[:2])
    bound = 2.0 * (2.0 ** -23 + np.sqrt(layer.oh * layer.ow / 32) * 2.0 ** -24)
    assert np.linalg.norm(gw[:2] - ref_w) < bound * np.linalg.norm(ref_w)
    assert not layer.pb or np.linalg.norm(gb[:2] - ref_b) < bound * np.linalg.norm(ref_b)
    assert np.allclose(sq[:2], ref_n2, rtol=2 * bound)


# Blocks that are larger than the chunks whose place in LDS they take, several examples per workgroup (the last one of fewer): one channel block and
# several, a chunk of two rows and of one.  Alone and in a batch call.
@pytest.mark.parametrize("cin,cout,h,w,n", [(128, 16, 2, 8, 1024), (256, 16, 2, 8, 515), (64, 16, 2, 2, 2049), (128, 9, 2, 7, 1030)])
@pytest.mark.parametrize("bias", [False, True])
def test_conv_f32_raw_rows_kernel_where_a_block_is_larger_than_its_chunks(cin, cout, h, w, n, bias):
    layer, few = Layer("conv", cin, cout, h, w, 5, 5, 1, 2, bias), 7
    x, dy = _inputs(layer, few, 151, "f32")
    ref_w, ref_b, ref_n2 = _oracle_grads(layer, x, dy)
    x, dy, ref_w, ref_b, ref_n2 = (np.resize(v, (n,) + v.shape[1:]) for v in (x, dy, ref_w, ref_b, ref_n2))
    assert dp.dp_kernel_variant(dp.make_desc(layer, n, "f32"), dp.DP_WS_PER_EXAMPLE_GRAD) == "conv_rows<f32,5x5,16x16,per_example>"
    gw, gb, sq = _run_per_example(layer, x, dy, "f32")
    xd, dyd, d = dev(x), dev(dy), dp.make_desc(layer, n, "f32")
    sizes = [dp.dp_workspace_bytes(d)] * 2
    wss = [torch.full((b,), 255, dtype=torch.uint8, device="cuda:0") for b in sizes]
    row, width = (layer.pw + 3) // 4 * 4, (layer.pw + 3) // 4 * 4 + (layer.pb + 3) // 4 * 4
    g = [torch.full((n, width), float("nan"), dtype=torch.float32, device="cuda:0") for _ in sizes]
    norms = torch.full((2, n), -1.0, device="cuda:0")
    batch = dp.LayerBatch([d, d], [t.data_ptr() for t in wss], sizes)
    dp.dp_per_example_grad_batch(batch, batch.ptrs([xd.data_ptr()] * 2), batch.ptrs([dyd.data_ptr()] * 2), batch.ptrs([t.data_ptr() for t in g]),
                                 batch.ptrs([t.data_ptr() + 4 * row for t in g]) if bias else None, batch.ptrs([v.data_ptr() for v in norms]), g_stride=width)
    torch.cuda.synchronize()
    for got_w, got_b, got_n2 in [(gw, gb, sq)] + [(host(t[:, :layer.pw]), host(t[:, row:row + layer.pb]), host(v)) for t, v in zip(g, norms)]:
        assert (np.linalg.norm(got_w - ref_w, axis=1) <= F32_TOL * np.linalg.norm(ref_w, axis=1)).all()
        assert not bias or (np.linalg.norm(got_b - ref_b, axis=1) <= F32_TOL * np.linalg.norm(ref_b, axis=1)).all()
        assert np.allclose(got_n2, ref_n2, rtol=F32_TOL, atol=0)


# ragged channels in one block and in several, rows of fewer than four numbers, no multiple of four and one column, both strides, two examples of a
# unit; several examples per workgroup
@pytest.mark.parametrize("cin,cout,h,w,k,stride,n,unit", [(33, 15, 27, 26, 3, 1, 300, 1), (18, 20, 45, 37, 5, 2, 40, 1), (18, 20, 40, 3, 3, 1, 300, 1), (17, 33, 30, 29, 3, 1, 300, 1),
                                                          (64, 32, 33, 34, 3, 2, 300, 1), (64, 64, 28, 28, 3, 1, 128, 2), (20, 40, 28, 27, 5, 1, 100, 1), (16, 16, 12, 14, 3, 1, 8200, 1)])
def test_conv_f32_raw_rows_kernel_computes_a_block_again(cin, cout, h, w, k, stride, n, unit):
    """Numbers whose parts are not finite while the sums of fp32 products are: every element within fp32 rounding of the sum of its products'
    magnitudes, in the broken examples and in the others."""
    layer, few = Layer("conv", cin, cout, h, w, k, k, stride, (k - 1) // 2, cout % 2 == 0), 4
    rng = np.random.default_rng(157)
    x, dy = _inputs(layer, few, 157, "f32")
    dy *= 2.0 ** -20
    for i, c in ((1, cin - 1), (2, 0)):
        x[i, c, rng.integers(h), rng.integers(w)], x[i, c, h - 1, w - 1] = np.finfo(np.float32).max, -np.finfo(np.float32).max
    name = dp.dp_kernel_variant(dp.make_desc(layer, n, "f32"), dp.DP_WS_PER_EXAMPLE_GRAD)
    assert name.startswith("conv_rows<f32"), name
    ref_w, ref_b, _ = _oracle_grads(layer, x, dy)
    abs_w, abs_b, _ = _oracle_grads(layer, np.abs(x), np.abs(dy))
    ref, mag = np.concatenate([ref_w, ref_b], axis=1), np.concatenate([abs_w, abs_b], axis=1)
    if unit > 1:
        ref, mag = ref.reshape(few // unit, unit, -1).sum(1), mag.reshape(few // unit, unit, -1).sum(1)
    rows = n // unit
    ref, mag, x, dy = np.resize(ref, (rows, ref.shape[1])), np.resize(mag, (rows, ref.shape[1])), np.resize(x, (n,) + x.shape[1:]), np.resize(dy, (n,) + dy.shape[1:])
    d = dp.make_desc(layer, n, "f32")
    need = dp.dp_unit_workspace_bytes(d, unit) if unit > 1 else dp.dp_workspace_bytes(d)
    ws, xd, dyd = torch.empty(max(16, need), dtype=torch.uint8, device="cuda:0"), dev(x), dev(dy)
    row = (layer.pw + 3) // 4 * 4
    g, sq = torch.full((rows, row + (layer.pb + 3) // 4 * 4), float("nan"), device="cuda:0"), torch.full((rows,), -1.0, device="cuda:0")
    args = (xd, dyd, g, g[:, row:] if layer.pb else None, sq, ws)
    dp.dp_unit_grad(d, unit, *args, g_stride=g.shape[1]) if unit > 1 else dp.dp_per_example_grad(d, *args, g_stride=g.shape[1])
    got = host(torch.cat([g[:, :layer.pw], g[:, row:row + layer.pb]], dim=1))
    assert (np.abs(got - ref) <= F32_TOL * mag).all(), np.abs(got / mag - ref / mag).max()


# The smallest numbers, whose parts end below the smallest ones of the narrower type: as exact as others.  (Gradients from 2^-90 on; the
# bound is that of test_conv_f32_raw_rows_kernel_is_as_exact_as_fp32.)
@pytest.mark.parametrize("up,down", [(60, 115), (0, 113), (-113, 0), (70, 130), (-45, 45), (90, 45)])
@pytest.mark.parametrize("cin,cout,h,w,k,stride,n", [(16, 16, 32, 32, 3, 1, 300), (40, 72, 45, 37, 5, 2, 40)])
def test_conv_f32_raw_rows_kernel_is_as_exact_on_small_numbers(cin, cout, h, w, k, stride, n, up, down):
    layer = Layer("conv", cin, cout, h, w, k, k, stride, (k - 1) // 2, k == 5)
    x, dy = _inputs(layer, 2, 163, "f32")
    x, dy = (x * 2.0 ** up).astype(np.float32), (dy * 2.0 ** -down).astype(np.float32)
    assert dp.dp_kernel_variant(dp.make_desc(layer, n, "f32"), dp.DP_WS_PER_EXAMPLE_GRAD).startswith("conv_rows<f32")
    ref_w = _oracle_grads(layer, x, dy)[0]
    gw = _run_per_example(layer, np.concatenate([x] * (n // 2)), np.concatenate([dy] * (n // 2)), "f32")[0]
    bound = 2.0 * (2.0 ** -23 + np.sqrt(layer.oh * layer.ow / 32) * 2.0 ** -24)
    scale = 2.0 ** (down - up)
    for got in (gw[:2], gw[-2:]):
        assert np.linalg.norm((got - ref_w) * scale) < bound * np.linalg.norm(ref_w * scale)


def test_conv_f32_raw_rows_kernel_takes_every_fp32_number():
    """Numbers that round to infinity as bf16 stay finite, NaNs stay where they are, and the next example is what it was."""
    layer = Layer("conv", 32, 16, 6, 8, 3, 3, 1, 1, False)
    x, dy = _inputs(layer, 400, 149, "f32")
    assert dp.dp_kernel_variant(dp.make_desc(layer, 400, "f32"), dp.DP_WS_PER_EXAMPLE_GRAD).startswith("conv_rows<f32")
    dy[:2] = 2.0 ** -20
    x[0, 3, 2, 4], x[1, 5, 0, 0] = np.finfo(np.float32).max, np.nan
    gw = _run_per_example(layer, x, dy, "f32")[0].reshape(400, 16, 32, 3, 3)
    ref = _oracle_grads(layer, x[[0, 2]], dy[[0, 2]])[0].reshape(2, 16, 32, 3, 3)
    assert_close(gw[0], ref[0], F32_TOL, "large numbers")
    assert_close(gw[2], ref[1], F32_TOL, "next example")
    want = np.zeros((3, 3), bool)                 # a corner: read by the taps at and left of and above the middle
    want[:2, :2] = True
    assert np.array_equal(np.isnan(gw[1, 0, 5]), want) and np.isfinite(np.delete(gw[1], 5, axis=1)).all()


# ---- clipping units in the kernels of the per-example calls: one unit (sliced into ranges of its examples), units no power of two,
# rows that end in a part chunk, enough units for the wide tile; every layer alone and all of one unit size in a batch call
_UNIT_ROUTES = [
    ("stem", conv(3, 64, 7, 2, 64), "bf16"), ("3x3 rows w56 sliced", conv(64, 64, 3, 1, 56), "bf16"), ("3x3 rows w14", conv(64, 70, 3, 1, 14), "bf16"),
    ("3x3 rows s2", conv(64, 64, 3, 2, 28), "bf16"), ("3x3 gather", conv(13, 70, 3, 1, 13), "bf16"), ("1x1 stride 2", conv(512, 256, 1, 2, 14), "bf16"),
    ("1x1 128x128 odd tail", conv(160, 136, 1, 1, 10), "bf16"), ("1x1 whole rows", conv(256, 512, 1, 1, 14), "bf16"),
    ("1x1 odd rows bias", conv(97, 71, 1, 1, 7, bias=True), "bf16"), ("fp32 5x5 stride 2", Layer("conv", 18, 20, 45, 37, 5, 5, 2, 2, True), "f32"),
]


@pytest.mark.parametrize("unit,units", [(4, 1), (3, 2), (2, 66)])
def test_units_in_the_per_example_kernels(unit, units):
    n = unit * units
    # 132 examples: the geometry with 256 x 128 tiles, whose rule asks for 128 of them
    cases = _UNIT_ROUTES if n < 100 else [("1x1 256x128", conv(256, 256, 1, 1, 10), "bf16"), ("1x1 whole rows", conv(256, 512, 1, 1, 14), "bf16")]
    runs = []
    for name, layer, dtype in cases:
        few = min(n, 2 * unit)                    # the oracle's few units, over and over
        x, dy = _inputs(layer, few, 139, dtype)
        mean_w, mean_b = oracle.unit_mean_grad(layer, x, dy, unit)
        xd, dyd = (dev(np.concatenate([v] * (n // few)), dtype) for v in (x, dy))
        d = dp.make_desc(layer, n, dtype)
        ws = torch.empty(max(16, dp.dp_unit_workspace_bytes(d, unit)), dtype=torch.uint8, device="cuda:0")
        row = (layer.pw + 3) // 4 * 4
        runs.append((name, layer, BF16_TOL if dtype == "bf16" else F32_TOL, mean_w, mean_b, xd, dyd, d, ws, row))
    for together in (False, True):
        for group in ([runs] if together else [[r] for r in runs]):
            gs = [torch.full((units, r[9] + (r[1].pb + 3) // 4 * 4), 7.0, device="cuda:0") for r in group]
            sq, norms = (torch.full((len(group), units), -1.0, device="cuda:0") for _ in range(2))
            for k, r in enumerate(group):
                batch = dp.LayerBatch([r[7]], [r[8].data_ptr()], [r[8].numel()])
                args = batch.ptrs([r[5].data_ptr()]), batch.ptrs([r[6].data_ptr()])
                if not together:
                    dp.dp_unit_grad(r[7], unit, r[5], r[6], gs[k], gs[k][:, r[9]:] if r[1].pb else None, sq[k], r[8], g_stride=gs[k].shape[1])
                dp.dp_unit_grad_batch(batch, unit, *args, None, None, batch.ptrs([norms[k].data_ptr()]))
            if together:
                batch = dp.LayerBatch([r[7] for r in group], [r[8].data_ptr() for r in group], [r[8].numel() for r in group])
                # one row length for all: the longest
                pitch = max(g.shape[1] for g in gs)
                gs = [torch.full((units, pitch), 7.0, device="cuda:0") for _ in group]
                dp.dp_unit_grad_batch(batch, unit, batch.ptrs([r[5].data_ptr() for r in group]), batch.ptrs([r[6].data_ptr() for r in group]),
                                      batch.ptrs([g.data_ptr() for g in gs]),
                                      batch.ptrs([g[:, r[9]:].data_ptr() if r[1].pb else None for g, r in zip(gs, group)]),
                                      batch.ptrs([sq[k].data_ptr() for k in range(len(group))]), g_stride=pitch)
            torch.cuda.synchronize()
            for k, (name, layer, tol, mean_w, mean_b, *_, row) in enumerate(group):
                g = host(gs[k]) / unit
                for u in range(units):
                    ref_w, ref_b = mean_w[u % len(mean_w)], mean_b[u % len(mean_w)] if layer.pb else None
                    assert_close(g[u, :layer.pw], ref_w, tol, f"{name} unit {u} dW")
                    if layer.pb:
                        assert_close(g[u, row:row + layer.pb], ref_b, tol, f"{name} unit {u} db")
                    n2 = oracle.sqnorm(ref_w) + (oracle.sqnorm(ref_b) if layer.pb else 0.0)
                    for got in (sq[k, u], norms[k, u]):
                        assert np.isclose(float(got) / unit ** 2, n2, rtol=tol), (name, u)


# the fp32 raw-row kernel adds a unit's examples to one block: units of two to four, one and several units per workgroup, tiles of
# channels that are not whole, both kernel sizes and strides (enough units that the kernel is chosen: it needs no more workspace than the
# partial norms of its blocks)
@pytest.mark.parametrize("cin,cout,h,w,k,stride,n,unit", [(16, 16, 16, 16, 3, 1, 600, 2), (33, 14, 12, 12, 3, 1, 300, 3), (20, 18, 9, 11, 3, 2, 800, 4),
                                                          (18, 20, 45, 37, 5, 2, 200, 2), (16, 16, 12, 14, 3, 1, 16600, 2)])
def test_units_in_the_fp32_raw_row_kernel(cin, cout, h, w, k, stride, n, unit):
    layer = Layer("conv", cin, cout, h, w, k, k, stride, (k - 1) // 2, cout % 2 == 0)
    d, units = dp.make_desc(layer, n, "f32"), n // unit
    blocks = -(-cout // 32) * -(-cin // (16 if k == 5 else 32))
    assert dp.dp_unit_workspace_bytes(d, unit) == (4 * units * blocks + 15) // 16 * 16
    x, dy = _inputs(layer, 2 * unit, 141, "f32")
    mean_w, mean_b = oracle.unit_mean_grad(layer, x, dy, unit)
    xd, dyd = (dev(v).repeat((n // (2 * unit),) + (1,) * (v.ndim - 1)).contiguous() for v in (x, dy))      # two units, over and over
    ws = torch.empty(dp.dp_unit_workspace_bytes(d, unit), dtype=torch.uint8, device="cuda:0")
    row = (layer.pw + 3) // 4 * 4
    g = torch.full((units, row + (layer.pb + 3) // 4 * 4), 7.0, device="cuda:0")
    sq, norms = torch.full((units,), -1.0, device="cuda:0"), torch.full((units,), -1.0, device="cuda:0")
    dp.dp_unit_grad(d, unit, xd, dyd, g, g[:, row:] if layer.pb else None, sq, ws, g_stride=g.shape[1])
    dp.dp_unit_grad(d, unit, xd, dyd, None, None, norms, ws)
    torch.cuda.synchronize()
    for u in range(2):
        assert torch.equal(g[u::2, :layer.pw], g[u, :layer.pw].expand(units // 2, -1)) and torch.equal(sq[u::2], sq[u].expand(units // 2))
        got = host(g[u]) / unit
        assert_close(got[:layer.pw], mean_w[u], F32_TOL, "dW")
        if layer.pb:
            assert_close(got[row:row + layer.pb], mean_b[u], F32_TOL, "db")
        n2 = oracle.sqnorm(mean_w[u]) + (oracle.sqnorm(mean_b[u]) if layer.pb else 0.0)
        assert np.isclose(float(sq[u]) / unit ** 2, n2, rtol=F32_TOL)
    assert np.allclose(host(norms), host(sq), rtol=F32_TOL)


# The bf16 raw-row 3x3 kernel where a workgroup makes several rows of results one after the other: the last group of them short, tiles of few
# channels, rows of 7 whose examples start between dwords (odd channels), one stage and several per example, pieces that an
# example's end cuts.  Alone, from 1024 blocks on; every gradient is compared with a batch call of two layers, whose plan is another one.
@pytest.mark.parametrize("cin,cout,h,w,stride,n", [(64, 64, 7, 7, 1, 1030), (65, 67, 7, 7, 1, 519), (64, 130, 9, 7, 1, 700), (72, 65, 14, 14, 1, 515),
                                                   (64, 64, 13, 14, 1, 1027), (64, 64, 8, 8, 1, 1538), (64, 64, 10, 16, 1, 1025), (64, 64, 14, 14, 2, 1029),
                                                   (128, 65, 28, 28, 2, 300), (64, 64, 5, 28, 1, 1026), (64, 65, 3, 56, 1, 600), (64, 64, 2, 32, 1, 1100)])
def test_conv3x3_rows_of_results_in_a_row(cin, cout, h, w, stride, n):
    layer = Layer("conv", cin, cout, h, w, 3, 3, stride, 1, False)
    d = dp.make_desc(layer, n, "bf16")
    assert dp.dp_kernel_variant(d, dp.DP_WS_PER_EXAMPLE_GRAD | dp.DP_VARIANT_MATERIALISE).startswith("conv3x3_rows")
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(331)
    x = torch.randn((n,) + tuple(layer.x_shape), generator=gen, device="cuda:0").bfloat16()
    dy = (torch.randn((n,) + tuple(layer.dy_shape), generator=gen, device="cuda:0") * 0.05).bfloat16()
    f32 = dict(dtype=torch.float32, device="cuda:0")

    def batch(count):
        ws = [torch.empty(max(16, dp.dp_workspace_bytes(d, dp.DP_WS_PER_EXAMPLE_GRAD)), dtype=torch.uint8, device="cuda:0") for _ in range(count)]
        g = [torch.full((n, (layer.pw + 3) & ~3), 7.0, **f32) for _ in range(count)]
        sq = [torch.full((n,), -1.0, **f32) for _ in range(count)]
        if count == 1:
            dp.dp_per_example_grad(d, x, dy, g[0], None, sq[0], ws[0], g_stride=g[0].shape[1])
        else:
            bt = dp.LayerBatch([d] * count, [t.data_ptr() for t in ws], [t.numel() for t in ws])
            dp.dp_per_example_grad_batch(bt, bt.ptrs([x.data_ptr()] * count), bt.ptrs([dy.data_ptr()] * count), bt.ptrs([t.data_ptr() for t in g]), None,
                                         bt.ptrs([t.data_ptr() for t in sq]), g_stride=g[0].shape[1])
        torch.cuda.synchronize()
        return [t[:, :layer.pw] for t in g], sq

    (g,), (sq,) = batch(1)
    (a, b), (sa, sb) = batch(2)
    assert torch.equal(a, b) and torch.equal(sa, sb)
    # the two plans add the same products in other orders: sums of at most 784 terms, sqrt(784) 2^-24 = 1.7e-6 of their size
    assert float((g - a).norm() / g.norm()) < 1e-5 and float((g - a).abs().max() / g.abs().max()) < 1e-5
    assert torch.allclose(sq, sa, rtol=1e-5)
    assert torch.allclose(sq, g.square().sum(1), rtol=1e-4)
    for i in (0, 1, n // 2, n - 2, n - 1):
        ref, _ = oracle.example_grad(layer, host(x[i]), host(dy[i]))
        assert_close(host(g[i]), ref.reshape(-1), F32_TOL, f"example {i}")        # (bf16 products are exact in fp32)


# The same for norms alone (up to sixteen rows in a row; 7 x 7 and 8 x 8: from products of rows, in another kernel), against the stored gradients
@pytest.mark.parametrize("cin,cout,h,w,stride,n", [(64, 64, 7, 7, 1, 1030), (64, 130, 9, 7, 1, 700), (72, 65, 14, 14, 1, 515), (64, 64, 13, 14, 1, 1027),
                                                   (64, 64, 10, 16, 1, 1025), (64, 64, 14, 14, 2, 1029), (64, 64, 5, 28, 1, 1026), (64, 64, 2, 32, 1, 1100)])
def test_conv3x3_norms_alone_of_rows_in_a_row(cin, cout, h, w, stride, n):
    layer = Layer("conv", cin, cout, h, w, 3, 3, stride, 1, False)
    d = dp.make_desc(layer, n, "bf16")
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(337)
    x = torch.randn((n,) + tuple(layer.x_shape), generator=gen, device="cuda:0").bfloat16()
    dy = (torch.randn((n,) + tuple(layer.dy_shape), generator=gen, device="cuda:0") * 0.05).bfloat16()
    ws = [torch.empty(max(16, dp.dp_workspace_bytes(d)), dtype=torch.uint8, device="cuda:0") for _ in range(2)]
    g, want = torch.empty((n, layer.pw), device="cuda:0"), torch.empty(n, device="cuda:0")
    dp.dp_per_example_grad(d, x, dy, g, None, want, ws[0])
    for count in (1, 2):
        sq = [torch.full((n,), -1.0, device="cuda:0") for _ in range(count)]
        bt = dp.LayerBatch([d] * count, [t.data_ptr() for t in ws[:count]], [t.numel() for t in ws[:count]])
        dp.dp_per_example_grad_batch(bt, bt.ptrs([x.data_ptr()] * count), bt.ptrs([dy.data_ptr()] * count), None, None, bt.ptrs([t.data_ptr() for t in sq]))
        torch.cuda.synchronize()
        for t in sq:
            assert torch.allclose(t, want, rtol=1e-3 if h * w <= 64 else 1e-5)
    assert torch.allclose(want, g.square().sum(1), rtol=1e-4)


# The clip-weighted form where a range holds more examples than a wave has lanes for factors, and where it ends inside a range
@pytest.mark.parametrize("cin,cout,h,w,n", [(320, 320, 7, 7, 1700), (64, 72, 14, 14, 131), (1024, 1024, 8, 8, 70), (65, 65, 7, 7, 67), (64, 64, 16, 28, 9)])
def test_conv3x3_weighted_ranges(cin, cout, h, w, n):
    layer = Layer("conv", cin, cout, h, w, 3, 3, 1, 1, False)
    d = dp.make_desc(layer, n, "bf16")
    assert dp.dp_kernel_variant(d, dp.DP_WS_RECOMPUTE).startswith("conv3x3_rows")
    x, dy = _inputs(layer, n, 337, "bf16")
    rng = np.random.default_rng(41)
    n2 = (rng.uniform(0.3, 2.5, n) ** 2).astype(np.float32)
    n2[0] = 0.0
    got, _ = _run_weighted(layer, x, dy, "bf16", n2, 1.0)
    f = np.array([oracle.clip_factor(float(v), 1.0) for v in n2])
    idx = rng.choice(layer.pw, size=2000, replace=False)
    assert_close(got[idx] - 1.0, oracle.weighted_sum_elems(layer, x, dy, f, idx), BF16_TOL, "increment")


# Packed operands taken through LDS: planes of odd size and odd channel counts (examples that start between dwords), ranges of examples that are
# no multiple of a workgroup's, channels that are none either, strides, taps with and without padding, a plane too large for it
@pytest.mark.parametrize("layer,n", [(conv(33, 70, 1, 1, 5), 19), (conv(65, 64, 1, 2, 13), 7), (conv(67, 65, 3, 2, 14), 37), (conv(513, 64, 3, 1, 4), 21),
                                     (conv(40, 33, 3, 1, 9), 5), (conv(64, 64, 3, 2, 8), 257), (Layer("conv", 12, 40, 11, 13, 5, 5, 2, 2, False), 6),
                                     (Layer("conv", 3, 40, 130, 140, 3, 3, 4, 1, False), 3), (Layer("conv", 31, 64, 1, 7, 3, 3, 1, 1, False), 18)],
                         ids=lambda v: str(v) if isinstance(v, int) else f"{v.cin}-{v.cout}-{v.kh}x{v.kw}s{v.stride}-{v.h}x{v.w}")
@pytest.mark.parametrize("several", [False, True])
def test_packed_operands(layer, n, several):
    x, dy = _inputs(layer, n, 347, "bf16")
    rng = np.random.default_rng(43)
    n2 = (rng.uniform(0.3, 2.5, n) ** 2).astype(np.float32)
    f = np.array([oracle.clip_factor(float(v), 1.0) for v in n2])
    idx = rng.choice(layer.pw, size=min(layer.pw, 3000), replace=False)
    ref = oracle.weighted_sum_elems(layer, x, dy, f, idx)
    if not several:
        got, _ = _run_weighted(layer, x, dy, "bf16", n2, 1.0)
    else:
        d = dp.make_desc(layer, n, "bf16")
        ws = [torch.empty(max(16, dp.dp_workspace_bytes(d, dp.DP_WS_RECOMPUTE)), dtype=torch.uint8, device="cuda:0") for _ in range(2)]
        acc = [torch.ones(layer.pw, device="cuda:0") for _ in range(2)]
        xd, dyd, sq = dev(x, "bf16"), dev(dy, "bf16"), dev(n2)
        bt = dp.LayerBatch([d, d], [t.data_ptr() for t in ws], [t.numel() for t in ws])
        dp.dp_clip_accumulate_recompute_batch(bt, bt.ptrs([xd.data_ptr()] * 2), bt.ptrs([dyd.data_ptr()] * 2), bt.ptrs([sq.data_ptr()] * 2), bt.floats([1.0, 1.0]),
                                              bt.ptrs([t.data_ptr() for t in acc]), bt.ptrs([None, None]))
        torch.cuda.synchronize()
        assert torch.equal(acc[0], acc[1])
        got = host(acc[0])
    assert_close(got[idx] - 1.0, ref, BF16_TOL, "increment")


def _check_packed(layer, n, several, x, dy):
    """The clip-weighted sum of the layer alone, or of two of it in a batch call, against the oracle; how many kernels that takes."""
    rng = np.random.default_rng(43)
    n2 = (rng.uniform(0.3, 2.5, n) ** 2).astype(np.float32)
    f = np.array([oracle.clip_factor(float(v), 1.0) for v in n2])
    idx = rng.choice(layer.pw, size=min(layer.pw, 3000), replace=False)
    ref = oracle.weighted_sum_elems(layer, x, dy, f, idx)
    d, count = dp.make_desc(layer, n, "bf16"), 2 if several else 1
    ws = [torch.empty(max(16, dp.dp_workspace_bytes(d, dp.DP_WS_RECOMPUTE)), dtype=torch.uint8, device="cuda:0") for _ in range(count)]
    acc = [torch.ones(layer.pw, device="cuda:0") for _ in range(count)]
    xd, dyd, sq = dev(x, "bf16"), dev(dy, "bf16"), dev(n2)
    bt = dp.LayerBatch([d] * count, [t.data_ptr() for t in ws], [t.numel() for t in ws])
    kernels = launches(lambda: dp.dp_clip_accumulate_recompute_batch(
        bt, bt.ptrs([xd.data_ptr()] * count), bt.ptrs([dyd.data_ptr()] * count), bt.ptrs([sq.data_ptr()] * count), bt.floats([1.0] * count),
        bt.ptrs([t.data_ptr() for t in acc]), bt.ptrs([None] * count)))
    assert torch.equal(acc[0], acc[-1])
    assert_close(host(acc[0])[idx] - 1.0, ref, BF16_TOL, "increment")
    return len(kernels)


# X taken through LDS, in a launch of its own, where the copies are large: planes of an odd size and odd channel counts, ranges of examples and
# channels that are no multiple of a workgroup's, planes that only just fit (one channel of one example a workgroup); from 24 MB on for a layer
# alone, 12 MB in a batch call
@pytest.mark.parametrize("layer,n", [(conv(67, 65, 3, 2, 14), 401), (conv(513, 64, 3, 1, 4), 181), (conv(40, 33, 3, 1, 9), 421), (Layer("conv", 12, 40, 11, 13, 5, 5, 2, 2, False), 907),
                                     (conv(64, 64, 3, 2, 8), 1501), (Layer("conv", 23, 40, 80, 101, 3, 3, 2, 1, False), 31), (Layer("conv", 7, 36, 127, 129, 3, 3, 3, 1, False), 111)],
                         ids=lambda v: str(v) if isinstance(v, int) else f"{v.cin}-{v.cout}-{v.kh}x{v.kw}s{v.stride}-{v.h}x{v.w}")
def test_packed_operands_through_lds(layer, n):
    x, dy = _inputs(layer, n, 347, "bf16")
    copy = 2 * n * layer.cin * layer.kh * layer.kw * ((layer.oh * layer.ow + 7) // 8 * 8)
    assert (24 << 20) <= copy <= (27 << 20)
    assert _check_packed(layer, n, False, x, dy) == 4                 # X, dY, the contraction, the sum over ranges
    half, third = -(-n // 2) + n // 100, n // 3                       # 12 MB a layer; less
    assert _check_packed(layer, half, False, x[:half], dy[:half]) == 3

    def ranges(examples):                                             # of a batch call of as little work as these
        return -(-examples * ((layer.oh * layer.ow + 7) // 8 * 8) // (512 if layer.cout > 64 else 2048))

    assert _check_packed(layer, half, True, x[:half], dy[:half]) == 3 + (ranges(half) > 1)
    assert _check_packed(layer, third, True, x[:third], dy[:third]) == 2 + (ranges(third) > 1)


def _weighted_batch(layers, n, seed=359):
    """A clip-weighted batch call of bf16 layers, and what it works on."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    descs = [dp.make_desc(l, n, "bf16") for l in layers]
    xs, dys = ([torch.randn((n,) + tuple(shape), generator=gen, device="cuda:0").bfloat16() for shape in shapes]
               for shapes in ([l.x_shape for l in layers], [l.dy_shape for l in layers]))
    ws = [torch.empty(max(16, dp.dp_workspace_bytes(d, dp.DP_WS_RECOMPUTE)), dtype=torch.uint8, device="cuda:0") for d in descs]
    sq = torch.rand(n, generator=gen, device="cuda:0") + 0.5
    acc = [torch.zeros(l.pw, device="cuda:0") for l in layers]
    bt = dp.LayerBatch(descs, [t.data_ptr() for t in ws], [t.numel() for t in ws])
    args = (bt, bt.ptrs([t.data_ptr() for t in xs]), bt.ptrs([t.data_ptr() for t in dys]), bt.ptrs([sq.data_ptr()] * len(layers)), bt.floats([1.0] * len(layers)),
            bt.ptrs([t.data_ptr() for t in acc]), bt.ptrs([None] * len(layers)))
    return (lambda: dp.dp_clip_accumulate_recompute_batch(*args)), (xs, dys, ws, sq, acc)


# Layers on 14 x 14 maps in batch calls whose rows travel in stages: norm-only (ranges of eight examples, the last one short; from 128 blocks on)
# and clip-weighted (one range; several of up to sixteen with a sum behind them), tiles of both matrices' directions, whole tensors and examples by address, an example
# that is left out
@pytest.mark.parametrize("cin,cout,n", [(256, 256, 131), (256, 512, 66), (512, 128, 67), (768, 384, 33), (1024, 256, 32), (256, 128, 1)])
@pytest.mark.parametrize("at", [False, True])
def test_row_stages(cin, cout, n, at):
    layer = conv(cin, cout, 1, 1, 14)
    d = dp.make_desc(layer, n, "bf16")
    # (one example is the other kernel's, whatever the call's work)
    assert dp.dp_kernel_variant(d, dp.DP_WS_RECOMPUTE | dp.DP_VARIANT_SHARED) == f"conv_contract<bf16,{'128x256rows' if n > 1 else '128x128'},weighted>"
    x, dy = _inputs(layer, n, 353, "bf16")
    if n > 40:
        dy[5] = 3e38                               # this example's gradient overflows: no number in its norm, nothing in the sum
    rng = np.random.default_rng(47)
    n2 = (rng.uniform(0.3, 2.5, n) ** 2).astype(np.float32)
    f = np.array([oracle.clip_factor(float(v), 1.0) for v in n2])
    if n > 40:
        n2[5], f[5] = np.inf, 0.0
    xd, dyd, sqd = dev(x, "bf16"), dev(dy, "bf16"), dev(n2)
    ws = [torch.empty(max(16, dp.dp_workspace_bytes(d, dp.DP_WS_RECOMPUTE), dp.dp_workspace_bytes(d)), dtype=torch.uint8, device="cuda:0") for _ in range(2)]
    sq = [torch.full((n,), -1.0, device="cuda:0") for _ in range(2)]
    acc = [torch.ones(layer.pw, device="cuda:0") for _ in range(2)]
    bt = dp.LayerBatch([d, d], [t.data_ptr() for t in ws], [t.numel() for t in ws])
    if at:
        tables = [torch.tensor([t.data_ptr() + i * t[0].numel() * 2 for i in range(n)], dtype=torch.int64, device="cuda:0") for t in (xd, dyd)]
        px, pdy = ([t.data_ptr()] * 2 for t in tables)
    else:
        px, pdy = [xd.data_ptr()] * 2, [dyd.data_ptr()] * 2
    dp.dp_per_example_grad_batch(bt, bt.ptrs(px), bt.ptrs(pdy), None, None, bt.ptrs([t.data_ptr() for t in sq]), addresses=at)
    dp.dp_clip_accumulate_recompute_batch(bt, bt.ptrs(px), bt.ptrs(pdy), bt.ptrs([sqd.data_ptr()] * 2), bt.floats([1.0, 1.0]),
                                          bt.ptrs([t.data_ptr() for t in acc]), bt.ptrs([None, None]), addresses=at)
    torch.cuda.synchronize()
    assert torch.equal(acc[0], acc[1])
    keep = [i for i in range(n) if f[i] != 0.0]
    g = np.stack([dy[i].reshape(cout, 196).astype(np.float64) @ x[i].reshape(cin, 196).astype(np.float64).T for i in keep])
    # fp32 sums of 196 products (sqrt(196) 2^-24 = 8e-7), of their squares and of at most 131 scaled blocks
    for t in sq:
        assert np.allclose(host(t)[keep], (g * g).sum((1, 2)), rtol=1e-5)
    assert_close(host(acc[0]) - 1.0, (f[keep][:, None, None] * g).sum(0).reshape(-1), 1e-5, "increment")


# The same in calls that fill the chip, of rows of 196 and of 204 values (where other waves issue the seventh load of a stage): norm-only (ranges of eight
# examples, the last one short; from 128 blocks on) and clip-weighted (one range; several of up to sixteen with a sum behind them; twelve examples and a
# call of enough work, which a third layer stands for), tiles of both matrices' directions, whole tensors and examples by address, an example that is left out
@pytest.mark.parametrize("cin,cout,n,hw", [(256, 256, 131, (14, 14)), (256, 512, 66, (14, 14)), (512, 128, 67, (14, 14)), (768, 384, 33, (14, 14)),
                                           (1024, 256, 32, (14, 14)), (256, 128, 1, (14, 14)), (256, 256, 12, (14, 14)), (256, 512, 65, (12, 17)), (512, 512, 19, (17, 12))])
@pytest.mark.parametrize("at", [False, True])
def test_row_stages_in_calls_that_fill_the_chip(cin, cout, n, hw, at):
    layer, filler = Layer("conv", cin, cout, *hw), conv(4096, 2048, 1, 1, 14)
    S = hw[0] * hw[1]
    d = dp.make_desc(layer, n, "bf16")
    rows = "128x256rows" in dp.dp_kernel_variant(d, dp.DP_WS_RECOMPUTE | dp.DP_VARIANT_SHARED)
    assert rows == (n >= 12)
    descs = [d, d, dp.make_desc(filler, n, "bf16")]
    x, dy = _inputs(layer, n, 353, "bf16")
    if n > 40:
        dy[5] = 3e38                               # this example's gradient overflows: no number in its norm, nothing in the sum
    rng = np.random.default_rng(47)
    n2 = (rng.uniform(0.3, 2.5, n) ** 2).astype(np.float32)
    f = np.array([oracle.clip_factor(float(v), 1.0) for v in n2])
    if n > 40:
        n2[5], f[5] = np.inf, 0.0
    xd, dyd, sqd = [dev(x, "bf16")] * 2, [dev(dy, "bf16")] * 2, dev(n2)
    xd.append(torch.ones((n,) + tuple(filler.x_shape), dtype=torch.bfloat16, device="cuda:0"))
    dyd.append(xd[2])
    ws = [torch.empty(max(16, dp.dp_workspace_bytes(e, dp.DP_WS_RECOMPUTE), dp.dp_workspace_bytes(e)), dtype=torch.uint8, device="cuda:0") for e in descs]
    sq = [torch.full((n,), -1.0, device="cuda:0") for _ in range(3)]
    acc = [torch.ones(p, device="cuda:0") for p in (layer.pw, layer.pw, filler.pw)]
    bt = dp.LayerBatch(descs, [t.data_ptr() for t in ws], [t.numel() for t in ws])
    if at:
        tables = [[torch.tensor([t.data_ptr() + i * t[0].numel() * 2 for i in range(n)], dtype=torch.int64, device="cuda:0") for t in ts] for ts in (xd, dyd)]
        px, pdy = ([t.data_ptr() for t in ts] for ts in tables)
    else:
        px, pdy = [t.data_ptr() for t in xd], [t.data_ptr() for t in dyd]

    def norms():
        dp.dp_per_example_grad_batch(bt, bt.ptrs(px), bt.ptrs(pdy), None, None, bt.ptrs([t.data_ptr() for t in sq]), addresses=at)

    def sums():
        dp.dp_clip_accumulate_recompute_batch(bt, bt.ptrs(px), bt.ptrs(pdy), bt.ptrs([sqd.data_ptr()] * 3), bt.floats([1.0] * 3),
                                              bt.ptrs([t.data_ptr() for t in acc]), bt.ptrs([None] * 3), addresses=at)

    norms()
    main = launches(sums)
    if rows:                                       # two layers of whole-row tiles, one workgroup a range of up to sixteen examples
        groups = (cout // 128) * (cin // 256) * -(-n // 16)
        assert 2 * -(-groups // 8) * 8 + 16 * 16 * min(-(-n // 16), 2) in main, (main, groups)        # (two copies of the third one's matrix are 67 MB)
    torch.cuda.synchronize()
    assert torch.equal(acc[0], acc[1])
    keep = [i for i in range(n) if f[i] != 0.0]
    g = np.stack([dy[i].reshape(cout, S).astype(np.float64) @ x[i].reshape(cin, S).astype(np.float64).T for i in keep])
    # fp32 sums of about 200 products (sqrt(204) 2^-24 = 9e-7), of their squares and of at most 131 scaled blocks
    for t in sq[:2]:
        assert np.allclose(host(t)[keep], (g * g).sum((1, 2)), rtol=1e-5)
    assert_close(host(acc[0]) - 1.0, (f[keep][:, None, None] * g).sum(0).reshape(-1), 1e-5, "increment")


# And where the call is too little for ranges of sixteen examples: the layers bring the workgroups that they bring in the other kernel
@pytest.mark.parametrize("cin,cout,count,n", [(256, 256, 2, 16), (512, 128, 4, 16), (256, 1024, 2, 32), (1024, 256, 2, 4)])
def test_row_stages_are_left_to_calls_that_fill_the_chip(cin, cout, count, n):
    call, _kept = _weighted_batch([conv(cin, cout, 1, 1, 14)] * count, n)
    assert launches(call)[0] >= 32 * count


# And taken where the other kernel leaves copies of small matrices to add, or few examples are ranges that the chip finishes at once
@pytest.mark.parametrize("cin,cout,count,n", [(256, 256, 6, 130), (256, 256, 8, 100), (256, 384, 16, 17), (2048, 384, 10, 7), (512, 256, 13, 20)])
def test_row_stages_are_taken_where_their_rounds_are_shorter(cin, cout, count, n):
    call, (xs, dys, _, sq, acc) = _weighted_batch([conv(cin, cout, 1, 1, 14)] * count, n)
    for t in acc:
        t.zero_()
    ranges = -(-n // 16)
    ranges = -(-n // -(-n // ranges))
    assert launches(call)[0] == count * -(-(cout // 128) * (cin // 256) * ranges // 8) * 8
    f = torch.clamp(1.0 / sq.double().sqrt(), max=1.0)
    for x, dy, got in ((xs[0], dys[0], acc[0]), (xs[-1], dys[-1], acc[-1])):
        x, dy = x.reshape(n, cin, 196)[:, :8].double(), dy.reshape(n, cout, 196).double() * f[:, None, None]
        assert_close(host(got.reshape(cout, cin)[:, :8]).reshape(-1), host(sum(dy[i] @ x[i].T for i in range(n))).reshape(-1), 1e-5, "sum")


# The ranges' copies of a matrix stay below 96 MB, the ranges get longer instead
def test_row_stages_keep_their_copies_small():
    layers = [conv(2048, 1024, 1, 1, 14), conv(512, 512, 3, 1, 14)]
    n = 240
    d = dp.make_desc(layers[0], n, "bf16")
    assert "128x256rows" in dp.dp_kernel_variant(d, dp.DP_WS_RECOMPUTE | dp.DP_VARIANT_SHARED)
    assert dp.dp_workspace_bytes(d, dp.DP_WS_RECOMPUTE) <= 96_000_000
    call, (xs, dys, _, sq, acc) = _weighted_batch(layers, n)
    for t in acc:
        t.zero_()
    assert 8 * 8 * 11 in launches(call)            # (fifteen ranges of sixteen would be 126 MB)
    f = torch.clamp(1.0 / sq.double().sqrt(), max=1.0)
    x, dy = xs[0].reshape(n, 2048, 196)[:, :8].double(), (dys[0].reshape(n, 1024, 196).double() * f[:, None, None])
    ref = sum(dy[i] @ x[i].T for i in range(n))
    assert_close(host(acc[0].reshape(1024, 2048)[:, :8]).reshape(-1), host(ref).reshape(-1), 1e-5, "sum")


# Steps of several micro-steps keep no gradients of such layers but the last one's: accumulator against single micro-steps, gradients of the last one whole
@pytest.mark.parametrize("streams", [1, 3])
def test_phases_that_others_follow(streams):
    from workloads.configs import Workload
    from workloads.device import make_device_inputs
    layers = (conv(64, 256, 1, 1, 14, name="a"), conv(256, 256, 1, 1, 14, name="b"), conv(256, 256, 3, 1, 14, name="c"), conv(1024, 256, 1, 1, 14, name="d"),
              dense(64, 12, name="fc"))
    wl = Workload("rows", layers, 130, 3, "bf16", "per_layer", 1.0, 0.0, tuple("abs" for _ in layers), 0.01, 77)
    inputs = make_device_inputs(wl, wl.accum, torch.device("cuda:0"))
    whole, single = (dp.PrivatiseStep(wl, streams=streams) for _ in range(2))
    assert whole.p_mat == single.p_mat and whole._plan(1, True).p_mat < whole.p_mat
    whole.run(inputs)
    single.begin_step()
    for step in inputs:
        single.micro_step(step)
    single.finalize()
    torch.cuda.synchronize()
    # the same blocks, squared and scaled in fp32 in another order
    assert_close(host(whole.acc), host(single.acc), 1e-5, "accumulator")
    assert_close(host(whole.group_sqnorm), host(single.group_sqnorm), 1e-5, "norms")
    assert torch.equal(whole.g, single.g)
    first = whole.acc.clone()
    whole.capture(inputs)
    for _ in range(3):
        whole.replay()
        torch.cuda.synchronize()
        assert torch.equal(whole.acc, first) and torch.equal(whole.g, single.g)


# The same with four such layers, and of a step that is broken off: accumulator against single micro-steps, gradients of the last one whole
@pytest.mark.parametrize("streams", [1, 3])
def test_phases_that_others_follow_broken_off_and_replayed(streams):
    from workloads.configs import Workload
    from workloads.device import make_device_inputs
    layers = (conv(64, 256, 1, 1, 14, name="a"), conv(256, 256, 1, 1, 14, name="b"), conv(256, 256, 3, 1, 14, name="c"), conv(1024, 256, 1, 1, 14, name="d"),
              conv(256, 1024, 1, 1, 14, name="e"), dense(64, 12, name="fc"))
    wl = Workload("rows", layers, 130, 3, "bf16", "per_layer", 1.0, 0.0, tuple("abs" for _ in layers), 0.01, 77)
    inputs = make_device_inputs(wl, wl.accum, torch.device("cuda:0"))
    whole, single = (dp.PrivatiseStep(wl, streams=streams) for _ in range(2))
    assert whole.p_mat == single.p_mat and whole._plan(1, True).p_mat < whole.p_mat
    whole.run(inputs)
    single.begin_step()
    for step in inputs:
        single.micro_step(step)
    single.finalize()
    torch.cuda.synchronize()
    # the same blocks, squared and scaled in fp32 in another order
    assert_close(host(whole.acc), host(single.acc), 1e-5, "accumulator")
    assert_close(host(whole.group_sqnorm), host(single.group_sqnorm), 1e-5, "norms")
    assert torch.equal(whole.g, single.g)
    first = whole.acc.clone()
    whole.capture(inputs)
    for _ in range(3):
        whole.replay()
        torch.cuda.synchronize()
        assert torch.equal(whole.acc, first) and torch.equal(whole.g, single.g)
    # broken off behind a phase that stored less
    with pytest.raises(IndexError):
        whole.run([*inputs[:2], []])
    single.begin_step()
    single.micro_step(inputs[1])
    torch.cuda.synchronize()
    assert whole.micro_steps_done == 2 and torch.equal(whole.g, single.g)


# The same with noise for every example, with momentum, with one bound for all layers, phases of several micro-steps whose last one is shorter, and steps of other
# lengths in between, against single micro-steps: the same blocks and the same deviates, added in another order
@pytest.mark.parametrize("n,together,noise,clip", [(140, 1, "per_example", "per_layer"), (60, 3, "once", "global"), (70, 2, "per_example", "global")])
@pytest.mark.parametrize("streams", [1, 4])
def test_phases_that_others_follow_in_steps_of_any_length(monkeypatch, n, together, noise, clip, streams):
    from workloads.configs import Workload
    from workloads.device import make_device_inputs
    layers = (conv(1024, 256, 1, 1, 14, name="a"), conv(64, 64, 3, 1, 14, name="b"), conv(256, 1024, 1, 1, 14, name="c"), gn_affine(32, 14, 4))
    wl = Workload("rows", layers, n, 5, "bf16", clip, 1.0, 0.5, tuple("normal" for _ in layers), 0.01, 79, philox_seed=5)
    inputs = make_device_inputs(wl, wl.accum, torch.device("cuda:0"))
    single = dp.PrivatiseStep(wl, noise=noise)
    monkeypatch.setattr(dp.PrivatiseStep, "_micro_steps_together", lambda self: together)
    whole = dp.PrivatiseStep(wl, streams=streams, noise=noise)
    assert whole._plan(together, True).form.count("recompute") >= 2 and whole._plan(together, True).p_mat < whole.p_mat
    for ps in (whole, single):
        ps.enable_update(lr=0.1, momentum=0.9)
    for length in (5, 2, 1, 5, 4):
        whole.run(inputs[:length])
        single.begin_step()
        for step in inputs[:length]:
            single.micro_step(step)
        single.finalize()
        torch.cuda.synchronize()
        assert torch.allclose(whole.g, single.g, rtol=1e-5, atol=1e-5 * float(single.g.abs().max()))
        for got, want, what in ((whole.acc, single.acc, "accumulator"), (whole.group_sqnorm, single.group_sqnorm, "norms"), (whole.out, single.out, "gradient"),
                                (whole.theta, single.theta, "parameters"), (whole.velocity, single.velocity, "momentum")):
            assert_close(host(got), host(want), 1e-5, f"{what}, {length} micro-steps")


# Packed layers whose copies are worth the launch through LDS together; three launches of copies and contraction, and one of sums over ranges
@pytest.mark.parametrize("layer,count,n", [(conv(290, 64, 3, 2, 18), 4, 16), (Layer("conv", 512, 64, 11, 64, 3, 3, 2, 1, False), 6, 4), (conv(64, 55, 5, 1, 25), 10, 3)],
                         ids=lambda v: str(v) if isinstance(v, int) else f"{v.cin}-{v.cout}-{v.kh}x{v.kw}s{v.stride}-{v.h}x{v.w}")
def test_packed_copies_of_several_layers_go_through_lds_together(layer, count, n):
    few, _few = _weighted_batch([layer] * 2, n)
    call, (xs, dys, _, sq, acc) = _weighted_batch([layer] * count, n)
    for t in acc:
        t.zero_()
    assert len(launches(call)) == len(launches(few)) + 1             # (two layers: all copies in one launch)
    f = torch.clamp(1.0 / sq.double().sqrt(), max=1.0)
    x, dy, got = xs[-1], dys[-1], acc[-1]
    scaled = (dy.double() * f[:, None, None, None]).float().bfloat16().double()
    ref = torch.nn.functional.unfold(x[:, :4].double(), layer.kh, padding=layer.pad, stride=layer.stride)
    ref = sum(scaled[i].reshape(layer.cout, -1) @ ref[i].T for i in range(n))
    assert_close(host(got.reshape(layer.cout, layer.cin, -1)[:, :4]).reshape(-1), host(ref).reshape(-1), 1e-4, "sum")


# The clip-weighted 3x3 form in batch calls: layers of few tiles still bring workgroups (up to what whole examples allow); in a full
# launch a tile is one workgroup, without slice sums
@pytest.mark.parametrize("layers,n,least", [([conv(64, 64, 3, 1, 14)] * 2, 48, 48), ([conv(64, 64, 3, 1, 28)] * 2, 32, 64), ([conv(64, 64, 3, 1, 7)] * 2, 128, 64),
                                            ([conv(256, 256, 3, 1, 14)] * 2, 48, 128), ([conv(128, 128, 3, 1, 28)] * 4, 16, 96)],
                         ids=lambda v: str(v) if isinstance(v, int) else f"{len(v)}x{v[0].cin}-{v[0].h}")
def test_conv3x3_weighted_batches_fill_the_chip(layers, n, least):
    call, (xs, dys, _, sq, acc) = _weighted_batch(layers, n)
    for t in acc:
        t.zero_()
    main = launches(call)[0]
    assert main >= least, main
    # recorded, not run: one call's sums, of which some are compared with products in fp64
    f = torch.clamp(1.0 / sq.double().sqrt(), max=1.0)
    for x, dy, got, l in zip(xs, dys, acc, layers):
        scaled = (dy.double() * f[:, None, None, None]).float().bfloat16().double()
        ref = torch.nn.functional.unfold(x[:, :4].double(), 3, padding=1)
        ref = sum(scaled[i].reshape(l.cout, -1) @ ref[i].T for i in range(n))
        assert_close(host(got.reshape(l.cout, l.cin, 9)[:, :4]).reshape(-1), host(ref).reshape(-1), 1e-4, "sum")


# The same beside a layer that another kernel runs, however much work that is, and on small maps (tiles x ranges of each such layer)
@pytest.mark.parametrize("layers,n,blocks", [([conv(256, 64, 3, 1, 7), conv(256, 256, 5, 1, 20)], 32, 4 * 8), ([conv(64, 64, 3, 1, 14), conv(512, 512, 5, 1, 14)], 48, 24),
                                             ([conv(193, 256, 3, 1, 7), conv(128, 128, 5, 1, 8)], 12, 16 * 2)],
                         ids=lambda v: str(v) if isinstance(v, int) else f"{v[0].cin}-{v[0].h}")
def test_conv3x3_weighted_layers_beside_other_kernels(layers, n, blocks):
    call, _kept = _weighted_batch(layers, n)
    assert blocks in launches(call)


# Stored and norm-only: a small launch keeps a workgroup per row of results, whatever else the call holds
def test_conv3x3_rows_of_a_small_launch_are_not_put_in_a_row():
    layers, n = [conv(512, 64, 3, 1, 8), conv(256, 256, 1, 1, 14)], 48
    descs = [dp.make_desc(l, n, "bf16") for l in layers]
    xs, dys = [torch.ones((n,) + tuple(l.x_shape), dtype=torch.bfloat16, device="cuda:0") for l in layers], [
        torch.ones((n,) + tuple(l.dy_shape), dtype=torch.bfloat16, device="cuda:0") for l in layers]
    ws = [torch.empty(max(16, dp.dp_workspace_bytes(d)), dtype=torch.uint8, device="cuda:0") for d in descs]
    g, sq = [torch.empty((n, l.pw), device="cuda:0") for l in layers], torch.zeros((2, n), device="cuda:0")
    bt = dp.LayerBatch(descs, [t.data_ptr() for t in ws], [t.numel() for t in ws])
    main = launches(lambda: dp.dp_per_example_grad_batch(bt, bt.ptrs([t.data_ptr() for t in xs]), bt.ptrs([t.data_ptr() for t in dys]), bt.ptrs([t.data_ptr() for t in g]), None,
                                                         bt.ptrs([sq[k].data_ptr() for k in range(2)])))
    assert 8 * n in main, main


def test_conv3x3_weighted_batches_of_a_full_launch_walk_one_range():
    layers = [conv(256, 256, 3, 1, 14)] * 5 + [conv(512, 512, 3, 1, 7)] * 2
    call, _kept = _weighted_batch(layers, 32)
    assert launches(call) == [5 * 16 + 2 * 64]


# Few large planes stay in the launch that packs both operands
@pytest.mark.parametrize("count", [1, 2])
def test_packed_planes_that_are_few_share_a_launch(count):
    layer, n = Layer("conv", 3, 64, 112, 112, 7, 7, 2, 3, False), 36
    call, _kept = _weighted_batch([layer] * count, n)
    assert launches(call)[0] > 10000               # a thread for every eight values of both operands
    assert len(launches(call)) == 3                # the contraction and the sum over ranges


# Ranges that fit the workspace are chosen for the shorter walk: four of six examples, a workgroup each (six of four would be three workgroups a tile)
def test_packed_ranges_leave_short_walks():
    call, _kept = _weighted_batch([Layer("conv", 64, 256, 56, 27, 3, 3, 1, 1, False), conv(512, 512, 3, 1, 30)], 24)
    assert 2 * 5 * 4 in launches(call)


# Packed operands in a batch call whose target makes ranges that the number of examples is no multiple of (here two of two for three examples):
# everything stays inside the workspace that was asked for
@pytest.mark.parametrize("layer,other,n", [(Layer("conv", 176, 64, 46, 46, 3, 3, 1, 1, False), conv(512, 512, 3, 1, 28), 3),
                                           (Layer("conv", 96, 64, 40, 44, 3, 3, 1, 1, False), conv(512, 512, 3, 1, 28), 5)], ids=["3", "5"])
def test_packed_operands_stay_in_the_workspace(layer, other, n):
    descs = [dp.make_desc(l, n, "bf16") for l in (layer, other)]
    need = [max(16, dp.dp_workspace_bytes(d, dp.DP_WS_RECOMPUTE)) for d in descs]
    guard = 16 << 20
    ws = [torch.full((b + guard,), 0x5A, dtype=torch.uint8, device="cuda:0") for b in need]
    ins = [_inputs(l, n, 367 + k, "bf16") for k, l in enumerate((layer, other))]
    xs, dys = [dev(x, "bf16") for x, _ in ins], [dev(dy, "bf16") for _, dy in ins]
    n2 = (np.random.default_rng(53).uniform(0.3, 2.5, n) ** 2).astype(np.float32)
    sq, acc = dev(n2), [torch.zeros(l.pw, device="cuda:0") for l in (layer, other)]
    bt = dp.LayerBatch(descs, [t.data_ptr() for t in ws], need)
    dp.dp_clip_accumulate_recompute_batch(bt, bt.ptrs([t.data_ptr() for t in xs]), bt.ptrs([t.data_ptr() for t in dys]), bt.ptrs([sq.data_ptr()] * 2),
                                          bt.floats([1.0, 1.0]), bt.ptrs([t.data_ptr() for t in acc]), bt.ptrs([None, None]))
    torch.cuda.synchronize()
    assert all(bool((t[b:] == 0x5A).all()) for t, b in zip(ws, need))
    f = np.array([oracle.clip_factor(float(v), 1.0) for v in n2])
    idx = np.random.default_rng(59).choice(layer.pw, size=1000, replace=False)
    assert_close(host(acc[0])[idx], oracle.weighted_sum_elems(layer, *ins[0], f, idx), BF16_TOL, "increment")


@pytest.mark.parametrize("count,n,rows", [(2, 48, 4), (1, 128, 4), (4, 8, 4), (1, 16, 2)])
def test_conv3x3_stored_rows_in_a_row_are_at_most_four(count, n, rows):
    layer = conv(512, 512, 3, 1, 7)
    d = dp.make_desc(layer, n, "bf16")
    x = torch.ones((n,) + tuple(layer.x_shape), dtype=torch.bfloat16, device="cuda:0")
    ws = [torch.empty(dp.dp_workspace_bytes(d), dtype=torch.uint8, device="cuda:0") for _ in range(count)]
    g, sq = torch.empty((n, layer.pw), device="cuda:0"), torch.zeros(n, device="cuda:0")
    bt = dp.LayerBatch([d] * count, [t.data_ptr() for t in ws], [t.numel() for t in ws])
    main = launches(lambda: dp.dp_per_example_grad_batch(bt, bt.ptrs([x.data_ptr()] * count), bt.ptrs([x.data_ptr()] * count), bt.ptrs([g.data_ptr()] * count), None,
                                                         bt.ptrs([sq.data_ptr()] * count)))[0]
    assert main == count * 64 * (n // rows)


# Values of X in the first and last row that are not finite stay with their example and their input channels
@pytest.mark.parametrize("w,stride", [(7, 1), (8, 1), (14, 1), (28, 1), (56, 1), (28, 2), (14, 2)])
def test_conv3x3_keeps_what_is_not_finite_in_its_example_and_channel(w, stride):
    layer, n, rng = conv(64, 64, 3, stride, w), 5, np.random.default_rng(61)
    x, dy = _inputs(layer, n, 373, "bf16")
    clean_w, _, clean_sq = _run_per_example(layer, x, dy, "bf16")
    for row, channel, value in ((0, 3, np.inf), (w - 1, 40, np.nan)):
        x[2, channel, row, rng.integers(w)] = value
    d = dp.make_desc(layer, n, "bf16")
    ws = torch.empty(dp.dp_workspace_bytes(d), dtype=torch.uint8, device="cuda:0")
    g, sq = torch.zeros((n, layer.pw), device="cuda:0"), torch.zeros(n, device="cuda:0")
    dp.dp_per_example_grad(d, dev(x, "bf16"), dev(dy, "bf16"), g, None, sq, ws)
    g, sq = g.cpu().numpy().reshape(n, 64, 64, 9), sq.cpu().numpy()
    keep = [0, 1, 3, 4]
    assert np.array_equal(g[keep], clean_w.reshape(n, 64, 64, 9)[keep]) and np.array_equal(sq[keep], clean_sq[keep]) and not np.isfinite(sq[2])
    others = [c for c in range(64) if c not in (3, 40)]
    assert np.array_equal(g[2][:, others], clean_w.reshape(n, 64, 64, 9)[2][:, others])
    # the centre row of taps reads both values; what does not read them is no number or what it was
    assert not np.isfinite(g[2][:, (3, 40), 3:6]).all(axis=(1, 2)).any()

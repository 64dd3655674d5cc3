"""GPU kernels at the edges of their tiles and of the rules that choose between them, against the oracle.

Tolerances: F32_TOL covers fp32 sums of up to a few thousand terms in any order (sqrt(K) 2^-24), BF16_TOL the one extra
rounding of scaled operands to bf16 (2^-9 per element)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2109_12191_amd as dp
from gpu_util import BF16_TOL, F32_TOL, assert_close, dev, host
from test_gpu_kernels import _inputs, _oracle_grads, _run_per_example
from workloads import dense, gn_affine, to_bf16_grid

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

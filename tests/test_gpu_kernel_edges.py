"""GPU kernels at the edges of their tiles and of the rules that choose between them, against the oracle.

Tolerances: F32_TOL covers fp32 sums of up to a few thousand terms in any order (sqrt(K) 2^-24), BF16_TOL the one extra
rounding of scaled operands to bf16 (2^-9 per element)."""
import numpy as np
import pytest

from gpu_util import BF16_TOL, F32_TOL, assert_close
from test_gpu_kernels import _inputs, _oracle_grads, _run_per_example
from workloads import gn_affine, to_bf16_grid

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


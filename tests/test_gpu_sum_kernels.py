"""Sum in the kernels whose operand is read at other times than the others': the resident kernel with 64-token tiles
(after its last step) and the persistent kernels with 5 and 6 step slots (in the post-operators, token counts that cut a
quad of tokens included), with weights that stay in registers and weights that are reloaded, one round of workgroups
and several."""
import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_parity import _run_sum, assert_parity

pytestmark = pytest.mark.gpu
TUNINGS = [(64, 101), (64, 102), (128, 16), (96, 16), (128, 112), (96, 112), (64, 112), (128, 108), (16, 106)]


@pytest.mark.parametrize("out_type", ["f32", "s8"])
@pytest.mark.parametrize("N,K,M,sparsity", [(400, 1024, 293, 0.82), (272, 1100, 387, 0.78), (144, 513, 130, 0.85), (1300, 300, 1601, 0.8)])
def test_sum_in_every_kernel_form(N, K, M, sparsity, out_type):
    case = wl.Case("sumk", N, K, M, sparsity, wl.N4K1, out_type, "none", keys=(97, N, K, M))
    d = wl.make(case)
    R = (wl.rng_for(98, N, M).standard_normal((N, M)) * wl.preact_sigma(K, case.sparsity)).astype(np.float32)
    ref = oracle.spmm(d["W"], d["X"], d["w_scale"], d["x_scale"], d["bias"], "none", out_type, d["out_scale"],
                      d["out_zero_point"], d["mid_scale"], d["x_zero_point"], sum=R)
    for i, tuning in enumerate(TUNINGS):
        assert_parity(_run_sum(d, case, R, M + i, tuning, i % 4), ref, case)

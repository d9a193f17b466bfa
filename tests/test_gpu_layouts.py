"""A sample's cost and variances do not depend on how many samples its block holds (16, 32 or 64) or
on the block's layout, bit for bit: the same samples in launches of 40, 4100 and 8200 samples, at the
points where the layout changes (row tiles in eights, LDS limits)."""
import numpy as np
import pytest

from paper_2411_03289_amd import gpmppi as B
from paper_2411_03289_amd import workloads as W

from gpu_util import dev, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["fp32", "bf16x3"])
@pytest.mark.parametrize("M", [256, 257, 300, 449, 512, 513, 576, 577, 700, 993, 1024])
def test_samples_do_not_depend_on_their_block(M, form):
    t = torch()
    got = []
    for K in (40, 4100, 8200):
        pr = W.small_problem(K=K, T=4, M=M, n_obs=5, path="eight", seed_data=610 + M % 7, U_scale=1.0,
                             n_data=max(M, 50))
        ctx = B.gpmppi_init(pr, B.FP32 if form == "fp32" else B.BF16X3)
        costs = t.empty(K, device="cuda")
        var = t.full((B.TRACE_SIZES["gp_var_d"](K, pr.T),), float("nan"), device="cuda")
        B.gpmppi_rollout(ctx, dev(pr.x0), dev(pr.U0), 77, costs, {"gp_var_d": var})
        t.cuda.synchronize()
        got.append((costs.cpu().numpy(), var.cpu().numpy().reshape(pr.T, 2, K)))
    for i in (0, 1):
        K = len(got[i][0])
        np.testing.assert_array_equal(got[i][0], got[i + 1][0][:K])
        np.testing.assert_array_equal(got[i][1], got[i + 1][1][:, :, :K])

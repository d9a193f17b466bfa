"""Launch shapes of a batch: two persistent workgroups per compute unit may be asked for wherever the
k operand of one output leaves room for them (whatever the kernels' own LDS plan holds), and the
results of the FP32 and BF16x3 forms do not depend on it."""
import numpy as np
import pytest

from paper_2411_03289_amd import gpmppi as B
from paper_2411_03289_amd import workloads as W

from gpu_util import dev, torch

pytestmark = pytest.mark.gpu


def _step(b, prs):
    t = torch()
    x0, U = dev(np.concatenate([p.x0 for p in prs])), dev(np.concatenate([p.U0.reshape(-1) for p in prs]))
    n = b.K_off[-1]
    out = [t.empty_like(U), t.empty(n, device="cuda"), t.empty(n, device="cuda")]
    B.gpmppi_batch_step(b, x0, U, 5, *out)
    t.cuda.synchronize()
    return [o.cpu().numpy() for o in out]


@pytest.mark.parametrize("form", ["fp32", "bf16x3"])
@pytest.mark.parametrize("M,groups", [(64, 1), (128, 1), (256, 1), (512, 1), (64, 2), (128, 2), (256, 2)])
def test_two_workgroups_per_compute_unit(M, groups, form):
    prs = [W.small_problem(K=K, T=3, M=M, n_obs=3, path="eight", seed_data=81 + K, U_scale=0.5, n_data=max(M, 50))
           for K in (33, 300)]
    b = B.gpmppi_batch_init(prs, B.FP32 if form == "fp32" else B.BF16X3)
    want = _step(b, prs)
    for wg, waves, order in ((2, 4, 0), (2, 8, 1), (1, 8, 0)):
        B.gpmppi_batch_set_tuning(b, groups, 0, wg, order, waves)
        assert B.gpmppi_batch_get_tuning(b)["wg_per_cu"] == wg
        for w, g in zip(want, _step(b, prs)):
            np.testing.assert_array_equal(w, g)


def test_two_workgroups_refused_without_room():
    prs = [W.small_problem(K=33, T=2, M=1024, n_obs=1, path="eight", seed_data=91, n_data=1024)]
    b = B.gpmppi_batch_init(prs, B.FP32)
    with pytest.raises(B.GpmppiError):
        B.gpmppi_batch_set_tuning(b, 1, 0, 2, 0, 8)

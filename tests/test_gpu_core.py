"""Block layouts of the FP32 and BF16x3 rollout at the edges of their ranges, against
the oracle at the bars of the parity tests: both outputs of a step in one phase with W
held in registers (up to 256 points) or streamed (16-sample blocks, up to 448 points),
and chunks of 256 points with 32 or 64 samples per block; ragged last blocks."""
import pytest

from oracle import mppi
from paper_2411_03289_amd import gpmppi as B
from paper_2411_03289_amd import workloads as W

from gpu_util import gpu_rollout
from test_gpu_parity import _bf16_bounds, _check_bf16_rollout, _check_rollout

pytestmark = pytest.mark.gpu

# M, K: 16-sample blocks up to 16 per compute unit (4096 samples), 32 up to 8192, then 64
CASES = [(32, 17), (33, 4097), (256, 1), (256, 4097), (257, 33), (448, 15), (449, 47), (512, 8193), (769, 33),
         (993, 8255), (1024, 65)]


@pytest.mark.parametrize("form", ["fp32", "bf16x3"])
@pytest.mark.parametrize("M,K", CASES)
def test_block_layouts_match_oracle(M, K, form):
    prec = B.FP32 if form == "fp32" else B.BF16X3
    pr = W.small_problem(K=K, T=3, M=M, n_obs=7, path="eight", seed_data=300 + M % 7, U_scale=1.0, n_data=max(M, 50))
    S_o, tr_o = mppi.rollout(pr, pr.x0, pr.U0, pr.seed)
    S_g, tr_g = gpu_rollout(pr, ctx=B.gpmppi_init(pr, prec))
    if prec == B.FP32:
        _check_rollout(pr, S_g, tr_g, S_o, tr_o, f"M={M} K={K}")
    else:
        _check_bf16_rollout(prec, S_g, tr_g, tr_o, _bf16_bounds(pr, tr_o), f"form={form} M={M} K={K}")

"""The gradient at the edges of its launches (32 points per row tile, 8 waves, 32 entries per
workgroup of the GP part, 64 samples per workgroup of the recursion, 128-blocks of the
length-scales' matrix part), and in chunks of samples, against the reference gradient at the
bars of the gradient's own tests."""
import numpy as np
import pytest

from paper_2411_03289_amd import gpmppi as B
from paper_2411_03289_amd import workloads as W

from gpu_util import dev, torch
from test_gpu_grad import _check, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,T,M", [(1, 1, 1), (31, 3, 32), (33, 2, 33), (65, 4, 128), (63, 3, 129), (64, 2, 257),
                                   (97, 2, 289), (40, 3, 385), (7, 2, 512)])
def test_gradient_at_launch_edges(K, T, M):
    pr = W.small_problem(K=K, T=T, M=M, n_obs=4, path="eight", seed_data=400 + M % 9, U_scale=1.0, n_data=max(M, 50))
    _check(pr, pr.seed, _run(pr, pr.seed, C=min(T, 2)), label=f"K={K} T={T} M={M}")


def test_chunks_of_samples_match_reference_gradient():
    """r alone (115 MB) fits the scratch array, r and the records do not: both entry points take the
    samples in two chunks."""
    pr = W.small_problem(K=4500, T=50, M=1, n_obs=1, path="circle", seed_data=71, U_scale=0.5)
    ctx = B.gpmppi_init(pr, B.FP32)
    got = _run(pr, pr.seed, C=10, ctx=ctx)
    _check(pr, pr.seed, got, label="two chunks")
    t = torch()
    out = [t.empty(n, device="cuda") for n in (1, 2 * pr.T, 8, 2, pr.K)]
    B.gpmppi_grad_noalloc(ctx, dev(pr.x0), dev(pr.U0), pr.seed, 0.05, 10, *out)
    t.cuda.synchronize()
    for a, b in zip(got, out):
        np.testing.assert_array_equal(b.cpu().numpy().reshape(-1), a.reshape(-1).astype(np.float32))

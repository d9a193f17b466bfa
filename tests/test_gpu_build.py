"""GP factorization on the device at the edges of its tiling (blocks of 32 points, jobs of
two by two blocks, four blocks of W per workgroup), against the oracle at the bars of the
parity tests."""
import numpy as np
import pytest

from oracle import gp as G
from paper_2411_03289_amd import gpmppi as B
from paper_2411_03289_amd import workloads as W

from test_gpu_parity import EPS32, _gp_case, _gpu_predict

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [2, 31, 32, 33, 64, 65, 97, 129, 161, 545, 1023])
def test_factorization_at_block_edges(M):
    pr, q = _gp_case(M)
    gm, gv = _gpu_predict(pr, q, B.FP32)
    for o, g in enumerate(G.build_pair(pr.Z, pr.y, pr.log_ell, pr.log_sf, pr.log_sn)):
        m, _, v = g.predict(q)
        absdot = np.abs(G.se_ard(q, g.Z, g.log_ell, g.log_sf)) @ np.abs(g.alpha)
        assert np.all(np.abs(gm[o] - m) <= 1e-5 + 8 * EPS32 * absdot)
        assert np.all(np.abs(gv[o] - v) <= 2e-6 + 1e-5 * v)

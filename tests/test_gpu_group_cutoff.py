"""Lane-group columns' positions with an active cutoff row, bit for bit (its
breakpoint is one FP64 quotient, sum and floor or ceiling like a row's)."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from test_gpu_groups import _instance
from test_gpu_parity import chap, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_degree,eq", [(1, 0.0), (2, 0.5), (5, 0.3), (13, 1.0), (26, 0.2)])
def test_positions_with_a_cutoff(chap, per_degree, eq):
    import torch

    mip = _instance(per_degree, per_degree, eq)
    P = oracle.OracleProblem(mip)
    G = chap.Problem(mip)
    for seed, cut in ((2, 3.0), (3, -40.0), (4, 0.3)):
        x = mipgen.random_point(mip, seed)
        x = np.where(mip.is_int == 1, x, np.round(x))
        w = mipgen.random_weights(P.mp + 1, seed + 3, wmax=6)
        say(f"group cutoff per_degree={per_degree} eq={eq} cut={cut}")
        xh, s = G.best_shift(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), cut)
        torch.cuda.synchronize()
        oxh, os_ = P.best_shift(x, w, cut)
        assert np.array_equal(s.cpu().numpy(), os_)
        assert np.array_equal(xh.cpu().numpy(), oxh)

"""Single calls on either side of the column count (2^19) from which the point
and the results move through two-pass permutations instead of one gather, and
at the permutations' chunk edges; with and without a cutoff row (whose
objective sum has a launch of its own), fractional and integral objectives.
Shifts, scores and jump values equal the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from test_gpu_parity import chap, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 257, (1 << 19) - 1, 1 << 19, (1 << 19) + 1, 65 * 8192 + 1])
def test_single_calls(chap, n):
    import torch

    mip = mipgen.random_mixed(40 + n % 7, n=n, m=1500, max_row_nnz=min(n, 9), frac_bin=0.5, frac_int=0.5, int_width=30)
    for frac in (False, True):
        if frac:
            mip.obj = mip.obj * 0.7   # c^T x then takes the exact accumulator
        P = oracle.OracleProblem(mip)
        G = chap.Problem(mip)
        x = mipgen.random_point(mip, 3)
        w = mipgen.random_weights(P.mp + 1, 4, wmax=5)
        xd, wd = torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda()
        for cut in (np.inf, float(mip.obj @ x) - 4.0):
            say(f"single calls n={n} frac={frac} cut={cut}")
            xh, s = G.best_shift(xd, wd, cut)
            jv, js = G.jump_values(xd, wd, cut)
            torch.cuda.synchronize()
            oxh, os_ = P.best_shift(x, w, cut)
            ojv, ojs = P.jump_values(x, w, cut)
            assert np.array_equal(s.cpu().numpy(), os_) and np.array_equal(xh.cpu().numpy(), oxh)
            assert np.array_equal(jv.cpu().numpy(), ojv) and np.array_equal(js.cpu().numpy(), ojs)

"""The move kernel where an iteration's rows take one workgroup, several, and
all of them: moves of columns around its 1024 threads and its wavefronts,
reweights over rows around its 4096 rows per workgroup, on integer data
(residuals updated) and fractional data (touched rows summed again). Walks
equal the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from test_gpu_parity import chap, compare_runs, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,deg,integer", [(50, 30, True), (4096, 1024, True), (4097, 1025, True), (9000, 8500, True),
                                           (60, 33, False), (4097, 1200, False), (9000, 8500, False)])
def test_moves_and_reweights(chap, m, deg, integer):
    mip = mipgen.random_mixed(900 + m + deg, n=120, m=m, max_row_nnz=4, frac_bin=0.3, frac_int=0.7 if integer else 0.4,
                              int_width=12, integer_data=integer, long_cols=6, long_deg=deg)
    P = oracle.OracleProblem(mip)
    for opts in (dict(), dict(rescore_cap=64)):
        G = chap.Problem(mip, **opts)
        say(f"step m={m} deg={deg} integer={integer} {opts}")
        # a long tenure leaves no admissible move after some iterations: reweights
        for iters, tenure, seed in ((60, 5, 3), (150, 200, 1)):
            g, o = G.tabu_run(iters, tenure, seed), P.tabu_run(iters, tenure, seed)
            if integer:
                compare_runs(g, o, f"m={m} deg={deg} tenure={tenure}")
            else:
                assert np.array_equal(g.trace["var"], o["trace"]["var"])
                assert np.array_equal(g.trace["viol"], o["trace"]["viol"])
                assert np.array_equal(g.resid[:-1], o["r"][:-1])
            assert tenure < 100 or np.any(o["trace"]["kind"] == 2)

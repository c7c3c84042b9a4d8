"""Moves whose rows are summed again (fractional data) by one workgroup of the move
kernel, two, many, and more rows than its most workgroups hold a wavefront for:
columns of 16 to 5000 entries, with more violated rows than a column can mend
(no scan for aspiration). Walks equal the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from test_gpu_parity import chap, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,deg", [(60, 16), (60, 17), (400, 33), (3000, 512), (9000, 4095), (9000, 4100), (20000, 9000)])
def test_rows_summed_again(chap, m, deg):
    mip = mipgen.random_mixed(31 + deg, n=30, m=m, max_row_nnz=2, frac_bin=0.4, frac_int=0.4, int_width=9,
                              integer_data=False, long_cols=12, long_deg=deg)
    P = oracle.OracleProblem(mip)
    o = P.tabu_run(40, 4, 3)
    for opts in (dict(), dict(rescore_cap=8)):
        say(f"rows summed again m={m} deg={deg} {opts}")
        g = chap.Problem(mip, **opts).tabu_run(40, 4, 3)
        for f in ("var", "viol", "x_new"):
            assert np.array_equal(g.trace[f], o["trace"][f]), f
        assert np.array_equal(g.resid[:-1], o["r"][:-1]) and np.array_equal(g.w, o["w"])

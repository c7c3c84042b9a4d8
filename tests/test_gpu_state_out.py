"""A finished walk's state in the caller's order (points by the column
permutation, residuals and weights of the normalised rows with the equality
rows' twins, the cutoff row): single walks, also read after their problem is
gone, and a batch of every size at once, against the oracle bit for bit. Sizes
around a workgroup, one column, one row, more rows than columns."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from test_gpu_parity import chap, compare_runs, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (3, 40), (255, 64), (256, 300), (257, 1), (1000, 1030)]


@pytest.mark.parametrize("iters", [0, 1, 60])
def test_state_out(chap, iters):
    mips = [mipgen.random_mixed(70 + k, n=n, m=m, max_row_nnz=min(6, n), int_width=9) for k, (n, m) in enumerate(SIZES)]
    refs = [oracle.OracleProblem(mip).tabu_run(iters, 5, 11 + k) for k, mip in enumerate(mips)]
    for k, mip in enumerate(mips):
        say(f"state out single {SIZES[k]} iters={iters}")
        G = chap.Problem(mip)
        run = G.tabu_run(iters, 5, 11 + k)
        del G
        compare_runs(run, refs[k], f"single {SIZES[k]}")
    say(f"state out batch iters={iters}")
    Gs = [chap.Problem(mip) for mip in mips]
    for k, run in enumerate(chap.batch_run(Gs, np.arange(len(mips)), 11 + np.arange(len(mips)), iters, 5)):
        compare_runs(run, refs[k], f"batch {SIZES[k]}")

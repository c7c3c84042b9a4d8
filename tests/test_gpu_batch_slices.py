"""Batches of row-staged walks: the record kernel's slices of a batch of at most
eight walks, and of more, are not those of a walk alone. Instances of one row
block and of two, with few and with tens of thousands of single-entry columns,
entries below a slice and over many: every walk equals the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from test_gpu_parity import chap, compare_runs, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

SIZES = [(300, 200, 2500), (6000, 3000, 60000), (3000, 9000, 120000), (40000, 9000, 90000)]


@pytest.mark.parametrize("walks", [2, 8, 9, 20])
def test_batch_slices(chap, walks):
    mips = [mipgen.powerlaw(k, n=n, m=m, nnz=nnz, cap=m // 3) for k, (n, m, nnz) in enumerate(SIZES)]
    refs = [oracle.OracleProblem(mip).tabu_run(15, 4, 7 + k) for k, mip in enumerate(mips)]
    problems = [chap.Problem(mip) for mip in mips]
    which = np.arange(walks) % len(SIZES)
    say(f"batch slices walks={walks}")
    for w, run in enumerate(chap.batch_run(problems, which, 7 + which, 15, 4)):
        compare_runs(run, refs[which[w]], f"walk {w} of {walks}, {SIZES[which[w]]}")

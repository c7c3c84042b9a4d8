"""Affected rescoring where every column is scored by lane groups: the scoring
launch also scans the kept scores of the other columns and records the best
moves. Column counts around a scanning workgroup's step and below one group, caps
that some lists exceed (those iterations score every column), infeasible starts
(reweights) and incumbents (pending copies): the walk equals the oracle's bit for
bit."""
from __future__ import annotations

import pytest

import mipgen
import oracle
from test_gpu_parity import chap, compare_runs, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(3, 2), (255, 100), (257, 300), (2049, 700), (9000, 4500)])
@pytest.mark.parametrize("cap", [1, 24, 1024])
def test_aff_scan(chap, n, m, cap):
    mip = mipgen.random_mixed(900 + n, n=n, m=m, max_row_nnz=min(6, n), int_width=12)
    G = chap.Problem(mip, rescore_cap=cap)
    P = oracle.OracleProblem(mip)
    for seed in (0, 1):
        say(f"aff scan n={n} m={m} cap={cap} seed={seed}")
        compare_runs(G.tabu_run(150, 6, seed), P.tabu_run(150, 6, seed), f"n={n} cap={cap} seed={seed}")

"""Sizes that take later rounds of loops which smaller tests run once: more than
4096 move records of unstaged columns, more than 524,288 scanned scores, results of
more than 64 MiB (and one walk of more than that), and single calls whose
permutations go through staging (more than 5 * 2^17 columns). Sparse instances; walks
and calls equal the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from test_gpu_parity import chap, compare_runs, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _sparse(seed, n, m, per_row=4):
    """Integers in [0, 9] and binaries, a few random columns per row."""
    rng = np.random.default_rng(seed)
    rows, cols = mipgen._distinct_per_group(rng, np.full(m, per_row), n)
    ub = np.where(rng.random(n) < 0.5, 1.0, 9.0)
    a = mipgen.coo_to_csr_csc(n, m, rows, cols, mipgen._signed_nonzero_ints(rng, rows.size, 9))
    sense = np.array([ord("L"), ord("G"), ord("E")], dtype=np.uint8)[rng.integers(0, 3, m)]
    return mipgen.MIP(n=n, m=m, csr_row_ptr=a[0], csr_col=a[1], csr_val=a[2], csc_col_ptr=a[3], csc_row=a[4],
                      csc_val=a[5], sense=sense, rhs=rng.integers(-9, 10, m).astype(float), lb=np.zeros(n), ub=ub,
                      is_int=np.ones(n, dtype=np.uint8), obj=rng.integers(-3, 4, n).astype(float))


@pytest.mark.parametrize("opts", [dict(), dict(row_stage=-1), dict(rescore_cap=64)])
def test_records_and_scans(chap, opts):
    mip = _sparse(1, 1_200_000, 30_000)
    say(f"many columns walk {opts}")
    compare_runs(chap.Problem(mip, **opts).tabu_run(6, 3, 5), oracle.OracleProblem(mip).tabu_run(6, 3, 5), str(opts))


def test_results_in_rounds(chap):
    mips = [_sparse(2, 1_000_000, 20_000), _sparse(3, 8_500_000, 500)]
    refs = [oracle.OracleProblem(mip).tabu_run(3, 3, 5 + k) for k, mip in enumerate(mips)]
    problems = [chap.Problem(mip) for mip in mips]
    for which in ([0] * 20, [0, 0, 1, 0, 1, 0]):   # 160 MB in three rounds; walks of 68 MB among walks of 8 MB
        which = np.array(which)
        say(f"results in rounds {len(which)} walks")
        for w, run in enumerate(chap.batch_run(problems, which, 5 + which, 3, 3)):
            compare_runs(run, refs[which[w]], f"walk {w} of {len(which)}")


@pytest.mark.parametrize("n", [524_289, 655_360, 655_361, 659_457, 1_100_003])
def test_staged_permutations(chap, n):
    import torch

    mip = _sparse(n, n, 40_000)
    P = oracle.OracleProblem(mip)
    G = chap.Problem(mip)
    for seed, cut in ((1, np.inf), (2, 100.0)):
        x = mipgen.random_point(mip, seed)
        w = mipgen.random_weights(P.mp + 1, seed)
        say(f"permutations n={n} cut={cut}")
        xh, s = G.best_shift(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), cut)
        torch.cuda.synchronize()
        oxh, os_ = P.best_shift(x, w, cut)
        assert np.array_equal(s.cpu().numpy(), os_) and np.array_equal(xh.cpu().numpy(), oxh)

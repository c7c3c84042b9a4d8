"""Iterations whose best move is tabu while few rows are violated (workgroup 0 of
the move kernel scans its column, then all workgroups share the application):
moves by aspiration, the best move that is not tabu instead, and reweights, on
small instances padded with rows that never bind, so that columns and rows ask
for one workgroup, a few, and many. Single walks, batches and proposal
iterations equal the oracle's."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from test_gpu_learned import compare_traces
from test_gpu_parity import chap, compare_runs, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _padded(seed, n, m, extra, deg, integer):
    """A small mixed instance with `extra` slack rows, `deg` of them in every column."""
    mip = mipgen.random_mixed(seed, n=n, m=m, max_row_nnz=4, frac_bin=0.6, frac_int=0.4, int_width=5)
    rng = np.random.default_rng(seed)
    rows = np.repeat(np.arange(m), np.diff(mip.csr_row_ptr))
    cols, more = mipgen._distinct_per_group(rng, np.full(n, deg), max(extra, 1))
    vals = rng.integers(1, 4, cols.size).astype(float) * (1.0 if integer else 0.7)
    r = np.concatenate([rows, m + more])
    c = np.concatenate([mip.csr_col.astype(np.int64), cols])
    v = np.concatenate([mip.csr_val, vals])
    a = mipgen.coo_to_csr_csc(n, m + extra, r, c, v)
    return mipgen.MIP(n=n, m=m + extra, csr_row_ptr=a[0], csr_col=a[1], csr_val=a[2], csc_col_ptr=a[3], csc_row=a[4],
                      csc_val=a[5], sense=np.concatenate([mip.sense, np.full(extra, ord("L"), dtype=np.uint8)]),
                      rhs=np.concatenate([mip.rhs, np.full(extra, 1e5)]), lb=mip.lb, ub=mip.ub, is_int=mip.is_int,
                      obj=mip.obj)


# base instances whose walks move by aspiration; slack rows, entries of a column in them
BASES = [(14, 20, 14, 15), (16, 30, 25, 15), (42, 12, 8, 8)]
PADS = [(0, 0), (4200, 40), (9000, 2500), (33000, 9000)]


@pytest.mark.parametrize("extra,deg", PADS)
@pytest.mark.parametrize("integer", [True, False])
def test_shared_application(chap, extra, deg, integer):
    aspired = reweighted = 0
    problems, refs = [], []
    for seed, n, m, tenure in BASES:
        mip = _padded(seed, n, m, extra, deg, integer)
        P = oracle.OracleProblem(mip)
        o = P.tabu_run(300, tenure, 1)
        for opts in (dict(), dict(row_stage=-1, chunk_min=2000), dict(rescore_cap=16)):
            G = chap.Problem(mip, **opts)
            say(f"shares seed={seed} extra={extra} deg={deg} integer={integer} {opts}")
            g = G.tabu_run(300, tenure, 1)
            if integer:
                compare_runs(g, o, f"seed={seed} extra={extra} deg={deg} {opts}")
            else:
                for f in ("var", "kind", "viol", "x_new", "score"):
                    assert np.array_equal(g.trace[f], o["trace"][f]), f
                assert np.array_equal(g.resid[:-1], o["r"][:-1]) and np.array_equal(g.w, o["w"])
        aspired += int(np.count_nonzero(o["trace"]["kind"] == 1))
        reweighted += int(np.count_nonzero(o["trace"]["kind"] == 2))
        problems.append(chap.Problem(mip))
        refs.append(P.tabu_run(100, 15, 1))
    assert reweighted > 100 and (aspired > 5 or not integer)
    say(f"shares batch extra={extra} deg={deg} integer={integer}")
    walks = np.arange(12) % len(BASES)
    for w, run in enumerate(chap.batch_run(problems, walks, np.ones(12, dtype=int), 100, 15)):
        for f in ("var", "kind", "viol", "score"):
            assert np.array_equal(run.trace[f], refs[walks[w]]["trace"][f]), (w, f)
        assert np.array_equal(run.w, refs[walks[w]]["w"])


@pytest.mark.parametrize("extra,deg", PADS)
def test_proposal_iterations(chap, extra, deg):
    for seed, n, m, tenure in BASES:
        mip = _padded(seed, n, m, extra, deg, True)
        G = chap.Problem(mip)
        say(f"shares learned seed={seed} extra={extra} deg={deg}")
        run = chap.learned_run(G, chap.Model(1), 200, tenure, 1, full_every=4, topk=max(2, n // 2), log_sets=1)
        ref = oracle.OracleProblem(mip).learned_replay(200, tenure, 1, 4, run.sets, run.set_offsets)
        compare_traces(run.trace, ref["trace"], f"seed={seed} extra={extra}")
        assert np.array_equal(run.x, ref["x"]) and np.array_equal(run.w, ref["w"])

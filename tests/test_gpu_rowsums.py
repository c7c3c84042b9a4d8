"""Residuals from scratch at the sizes where their kernels split the work.

Integer data: the x-block kernel's workgroups own 64..4096 rows, chosen from
the row count and the chip's compute units. Other data: rows of more than 32
entries are summed by a wavefront, 256 entries per round, the rest by eight
lanes; a move's rows likewise. Every sum keeps the row's stored order, so
results equal the oracle's bit for bit.
"""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from helpers import make_mip
from test_gpu_parity import chap, compare_runs, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(17, 1), (15, 63), (33, 64), (100, 65), (2001, 16384), (500, 16385), (4097, 33001)])
def test_x_block_row_groups(chap, n, m):
    import torch

    mip = mipgen.random_mixed(n + m, n=n, m=m, max_row_nnz=7, frac_bin=0.4, frac_int=0.6, int_width=30)
    P = oracle.OracleProblem(mip)
    G = chap.Problem(mip)
    x = mipgen.random_point(mip, 3)
    w = mipgen.random_weights(P.mp + 1, 4, wmax=5)
    say(f"best_shift n={n} m={m}")
    xh, s = G.best_shift(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda())
    torch.cuda.synchronize()
    oxh, os_ = P.best_shift(x, w)
    assert np.array_equal(s.cpu().numpy(), os_) and np.array_equal(xh.cpu().numpy(), oxh)
    compare_runs(G.tabu_run(6, 5, 2), P.tabu_run(6, 5, 2), f"n={n} m={m}")


@pytest.mark.parametrize("fractional", [True, False])
def test_long_rows_in_stored_order(chap, fractional):
    """Rows of 1 .. 700 entries around the wavefront's limits (32 | 33, one
    and two rounds), with magnitudes that make every other order of summation
    visible in the last bits when the data are fractional."""
    rng = np.random.default_rng(5)
    n, lens = 800, [1, 8, 31, 32, 33, 40, 63, 64, 65, 128, 255, 256, 257, 300, 511, 512, 513, 700]
    rows = []
    for k, ln in enumerate(lens):
        cols = rng.choice(n, size=ln, replace=False)
        a = rng.uniform(-1, 1, ln) * 10.0 ** rng.integers(-3, 4, ln) if fractional else rng.integers(1, 9, ln)
        rows.append(({int(c): float(v) for c, v in zip(cols, a)}, "LGE"[k % 3], float(rng.integers(-40, 40))))
    # wide integers and continuous variables: no byte copy of x
    is_int = rng.integers(0, 2, n) if fractional else np.ones(n, dtype=int)
    mip = make_mip(n, rows, np.full(n, -300.0), np.full(n, 300.0), is_int, rng.integers(-3, 4, n))
    P = oracle.OracleProblem(mip)
    G = chap.Problem(mip)
    for iters, seed in ((0, 3), (1, 3), (40, 4)):
        say(f"long rows fractional={fractional} iters={iters}")
        g, o = G.tabu_run(iters, 5, seed), P.tabu_run(iters, 5, seed)
        assert np.array_equal(g.resid[:-1], o["r"][:-1])
        assert np.array_equal(g.trace["var"], o["trace"]["var"])
        assert np.array_equal(g.trace["x_new"], o["trace"]["x_new"])

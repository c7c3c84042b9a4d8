"""Lane-group scoring (columns of at most 64 stored entries outside the staged
tasks) at the edges of its widths: column degrees around 4, 8, 16, 32 and 64,
every variable type, equality rows (two terms per entry), infinite bounds, an
active cutoff row, column counts that leave the last workgroup and the last
group ragged. Scores and positions equal the oracle's bit for bit."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from helpers import make_mip
from test_gpu_parity import chap, compare_runs, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

DEGREES = [0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 70]


def _instance(seed, per_degree, eq):
    """per_degree columns of each degree and type over 160 rows."""
    rng = np.random.default_rng(seed)
    m, rows, lb, ub, is_int = 160, [dict() for _ in range(160)], [], [], []
    j = 0
    for d in DEGREES:
        for k in range(per_degree):
            for r in rng.choice(m, size=d, replace=False):
                rows[r][j] = int(rng.integers(1, 10)) * (1 if rng.random() < 0.5 else -1)
            kind = k % 5   # binary, narrow integer, wide integer, continuous, unbounded
            lb.append([0, -3, 0, 0, -np.inf][kind])
            ub.append([1, 20, 300, 50, np.inf][kind])
            is_int.append([1, 1, 1, 0, 1][kind])
            j += 1
    sense = rng.choice(["L", "G", "E"], size=m, p=[(1 - eq) / 2, (1 - eq) / 2, eq])
    listed = [(rows[i], sense[i], int(rng.integers(-60, 60))) for i in range(m)]
    return make_mip(j, listed, np.array(lb), np.array(ub), np.array(is_int), rng.integers(-4, 5, j))


@pytest.mark.parametrize("per_degree,eq", [(1, 0.0), (2, 0.5), (5, 0.3), (13, 1.0), (26, 0.2)])
def test_group_widths(chap, per_degree, eq):
    import torch

    mip = _instance(per_degree, per_degree, eq)
    P = oracle.OracleProblem(mip)
    G = chap.Problem(mip)
    R = chap.Problem(mip, rescore_cap=64)
    for seed, cut in ((1, np.inf), (2, 3.0), (3, -40.0)):
        x = mipgen.random_point(mip, seed)
        x = np.where(mip.is_int == 1, x, np.round(x))   # integer residuals: ties are exact
        w = mipgen.random_weights(P.mp + 1, seed + 3, wmax=6)
        say(f"group widths per_degree={per_degree} eq={eq} cut={cut}")
        xh, s = G.best_shift(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), cut)
        torch.cuda.synchronize()
        oxh, os_ = P.best_shift(x, w, cut)
        assert np.array_equal(s.cpu().numpy(), os_)
        assert np.allclose(xh.cpu().numpy(), oxh, rtol=1e-12, atol=0) if np.isfinite(cut) else np.array_equal(
            xh.cpu().numpy(), oxh)
    ref = P.tabu_run(40, 5, 4)
    for what, H in (("full", G), ("affected", R)):
        say(f"group widths walk {what}")
        g = H.tabu_run(40, 5, 4)
        assert np.array_equal(g.trace["var"], ref["trace"]["var"])
        assert np.array_equal(g.trace["score"], ref["trace"]["score"])

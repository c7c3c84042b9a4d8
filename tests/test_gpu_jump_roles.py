"""Jump values at the edges of the scoring roles: columns of 0, 1, 2, 7, 8, 9,
64, 65 and 1030 entries of every variable type, counts that leave the last lane
group and workgroup ragged, coefficients within and beyond [-127, 127] (both
quotients of the bins), integer and fractional weights (exact data or not),
with and without an acting cutoff row. Values and scores equal the oracle's bit
for bit: every column is one chunk, summed in the oracle's order, and the bins'
integer sums are exact."""
from __future__ import annotations

import math

import numpy as np
import pytest

import mipgen
import oracle
from helpers import make_mip
from test_gpu_jump import check_exact
from test_gpu_parity import chap, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

DEGREES = [0, 1, 2, 7, 8, 9, 64, 65, 1030]


def _instance(seed, per_degree, amax):
    rng = np.random.default_rng(seed)
    m, lb, ub, is_int = 1100, [], [], []
    rows = [dict() for _ in range(m)]
    j = 0
    for d in DEGREES:
        for k in range(per_degree):
            for r in rng.choice(m, size=d, replace=False):
                rows[r][j] = int(rng.integers(1, amax + 1)) * (1 if rng.random() < 0.5 else -1)
            kind = k % 5   # binary, narrow integer, 64 values, wide integer, continuous
            lb.append([0, -3, -30, 0, 0][kind])
            ub.append([1, 20, 33, 300, 50][kind])
            is_int.append([1, 1, 1, 1, 0][kind])
            j += 1
    sense = rng.choice(["L", "G", "E"], size=m, p=[0.4, 0.3, 0.3])
    listed = [(rows[i], sense[i], int(rng.integers(-60, 60))) for i in range(m)]
    return make_mip(j, listed, np.array(lb), np.array(ub), np.array(is_int), rng.integers(-4, 5, j))


@pytest.mark.parametrize("per_degree,amax", [(1, 1), (5, 9), (5, 127), (5, 128), (7, 3000), (33, 20)])
def test_jump_roles(chap, per_degree, amax):
    mip = _instance(per_degree + amax, per_degree, amax)
    P = oracle.OracleProblem(mip)
    G = chap.Problem(mip)
    for seed in (1, 2):
        x = mipgen.random_point(mip, seed)
        xi = np.where(mip.is_int == 1, x, np.round(x))
        w = mipgen.random_weights(P.mp + 1, seed, wmax=9)
        half = (w * np.float32(0.5)).astype(np.float32)
        for name, xx, ww in (("integers", xi, w), ("continuous point", x, w), ("half weights", xi, half)):
            for cut in (math.inf, P.objective(xx) - 3.0, P.objective(xx) + 40.0):
                say(f"jump roles per_degree={per_degree} amax={amax} seed={seed} {name} cutoff={cut}")
                check_exact(chap, mip, xx, ww, cut, f"{name} {seed}", G)

"""Row-block staging's record formats: coefficients at and beyond the int8 edge
(4-byte entries and float quotients up to 127, 8-byte entries and FP64 quotients
beyond), bounds beyond int16, one and several row blocks, widths up to 64
values, fractional and wide weights, with and without the cutoff row. Passes
and walks equal the oracle's and the unstaged form's."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from test_gpu_parity import chap, compare_runs, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _shifted(mip, by):
    """The same instance with every variable moved by `by`."""
    ones = np.zeros(mip.m)
    np.add.at(ones, np.repeat(np.arange(mip.m), np.diff(mip.csr_row_ptr)), mip.csr_val)
    mip.lb = mip.lb + by
    mip.ub = mip.ub + by
    mip.rhs = mip.rhs + by * ones
    return mip


@pytest.mark.parametrize("amax,umax,m,shift", [(9, 50, 3000, 0), (127, 63, 17000, 0), (128, 63, 17000, 0),
                                               (4000, 7, 9000, 0), (1, 1, 900, 0), (9, 50, 9000, 40000),
                                               (127, 63, 8192, -30000), (126, 40, 8193, -33000)])
def test_stage_records(chap, amax, umax, m, shift):
    import torch

    mip = mipgen.powerlaw(amax + m, n=6000, m=m, nnz=70_000, cap=min(m, 3000), umax=umax, amax=amax)
    if umax == 1:
        mip.ub = mip.ub + 1   # not binaries: narrow columns of three values
    mip = _shifted(mip, float(shift))
    P = oracle.OracleProblem(mip)
    G = chap.Problem(mip, chunk_min=900, chunk_len=128)
    for seed, wmax, scale, cut in ((1, 6, 1.0, np.inf), (2, 60000, 1.0, np.inf), (3, 6, 0.25, np.inf),
                                   (4, 6, 1.0, float(round(float(mip.obj @ mip.lb))))):
        x = mipgen.random_point(mip, seed)
        w = (mipgen.random_weights(P.mp + 1, seed + 5, wmax=wmax) * scale).astype(np.float32)
        say(f"stage records amax={amax} umax={umax} m={m} shift={shift} wmax={wmax} scale={scale}")
        xh, s = G.best_shift(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), cut)
        torch.cuda.synchronize()
        oxh, os_ = P.best_shift(x, w, cut)
        assert np.array_equal(s.cpu().numpy(), os_) and np.array_equal(xh.cpu().numpy(), oxh)
    compare_runs(G.tabu_run(25, 5, 3), P.tabu_run(25, 5, 3), f"amax={amax} m={m}")

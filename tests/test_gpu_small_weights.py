"""Best shifts with weights of every size a float holds, subnormal ones among
them (odd multiples of 2^-149, whose half is no float): scores are sums of
weights and half weights in FP64, and with weights that are small multiples of
one power of two every sum is exact, so they equal the oracle's bit for bit. The
row-staged, chunked, packed, sorted and lane-group columns take the same data."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from test_gpu_parity import chap, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("unit", [2.0 ** -149, 2.0 ** -126, 2.0 ** -1, 2.0 ** 120])
@pytest.mark.parametrize("kind", ["mixed", "long", "staged"])
def test_weight_units(chap, unit, kind):
    import torch

    mip = {"mixed": lambda: mipgen.random_mixed(5, n=400, m=300, max_row_nnz=8, int_width=200),
           "long": lambda: mipgen.random_mixed(6, n=60, m=900, max_row_nnz=4, int_width=40, long_cols=20, long_deg=300),
           "staged": lambda: mipgen.powerlaw(3, n=400, m=300, nnz=4000, cap=200)}[kind]()
    P = oracle.OracleProblem(mip)
    for opts in (dict(), dict(row_stage=-1), dict(chunk_min=64, chunk_len=64)):
        G = chap.Problem(mip, **opts)
        for seed, cut in ((1, np.inf), (2, 3.0)):
            x = mipgen.random_point(mip, seed)
            x = np.where(mip.is_int == 1, x, np.round(x))
            w = (mipgen.random_weights(P.mp + 1, seed, wmax=7).astype(np.float64) * unit).astype(np.float32)
            say(f"weights unit={unit} kind={kind} {opts} cut={cut}")
            xh, s = G.best_shift(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), cut)
            torch.cuda.synchronize()
            oxh, os_ = P.best_shift(x, w, cut)
            assert np.array_equal(s.cpu().numpy(), os_)
            assert np.array_equal(xh.cpu().numpy(), oxh)

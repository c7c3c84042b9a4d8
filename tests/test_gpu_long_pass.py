"""Single passes over columns sorted in global memory, which run on a stream of
the problem's own beside the others: calls queued one after another on the
caller's stream, with other points, weights and cutoffs and without a
synchronisation between them, equal the oracle's, also when the problem is
released right after the last call."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
import oracle
from test_gpu_parity import chap, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frac_int", [0.2, 0.6])
def test_queued_calls(chap, frac_int):
    import torch

    # columns of 4,500 entries: continuous ones and wide integers are sorted, narrow ones chunked
    mip = mipgen.random_mixed(12, n=300, m=5000, max_row_nnz=5, frac_bin=0.2, frac_int=frac_int, int_width=100,
                              long_cols=12, long_deg=4500)
    P = oracle.OracleProblem(mip)
    G = chap.Problem(mip, chunk_min=1000)
    stream = torch.cuda.Stream()
    calls = []
    for seed in range(5):
        x = mipgen.random_point(mip, seed)
        x = np.where(mip.is_int == 1, x, np.round(x))
        w = mipgen.random_weights(P.mp + 1, seed + 7)
        calls.append((x, w, np.inf if seed % 2 else 5.0 * seed))
    dev = [(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda(), cut) for x, w, cut in calls]
    torch.cuda.synchronize()
    say(f"queued passes frac_int={frac_int}")
    outs = [G.best_shift(x, w, cut, stream=stream) for x, w, cut in dev]
    del G
    stream.synchronize()
    for (x, w, cut), (xh, s) in zip(calls, outs):
        oxh, os_ = P.best_shift(x, w, cut)
        assert np.array_equal(s.cpu().numpy(), os_)
        assert np.array_equal(xh.cpu().numpy(), oxh)

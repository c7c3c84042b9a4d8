"""The no-allocation call at its scratch limit: a row-staged problem whose
entries fill it to the last few kilobytes, where the padding of the staged
records to whole pairs would pass it. The call takes it, and the single records
that its kernels then read give the results of the unstaged kernels, also in
walks and in a batch beside a problem with pairs."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
from test_gpu_parity import chap, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

LIMIT = 64 << 20


def _instance(n, m, entries, seed=1):
    """Integers in [0, 50], `entries` of them spread evenly over the columns."""
    rng = np.random.default_rng(seed)
    deg = np.full(n, entries // n)
    deg[: entries - deg.sum()] += 1
    cols, rows = mipgen._distinct_per_group(rng, deg, m)
    vals = mipgen._signed_nonzero_ints(rng, rows.shape[0], 9)
    hidden = rng.integers(0, 51, n).astype(float)
    sense = np.where(rng.random(m) < 0.05, ord("E"), ord("L"))
    return mipgen._finish(n, m, rows, cols, vals, sense, lambda act: act + 0.0, np.zeros(n), np.full(n, 50.0),
                          np.ones(n), rng.integers(-5, 6, n).astype(float), hidden, "limit")


def test_records_fill_the_scratch(chap):
    import torch

    assert chap.load_library().chap_best_shift_noalloc_max_bytes() == LIMIT
    n, m = 200_000, 245_760
    # per variable three doubles and a byte, per row 24 bytes, an 8-byte record per entry, the set-up's
    # 140 kB of partial sums and a few kilobytes of records and alignment
    left = LIMIT - 25 * n - 24 * m - 17_920 * 8 - 30_000
    mip = _instance(n, m, left // 8)
    G, U = chap.Problem(mip), chap.Problem(mip, row_stage=-1)
    for quarter in (False, True):
        x = torch.from_numpy(mipgen.random_point(mip, 2)).cuda()
        w = mipgen.random_weights(G.mp + 1, 3) + (0.25 if quarter else 0.0)
        w = torch.from_numpy(w.astype(np.float32)).cuda()
        for cut in (np.inf, 3.0):
            say(f"scratch limit quarter={quarter} cut={cut}")
            out = torch.empty_like(x), torch.empty_like(x)
            G.best_shift_noalloc(x, w, *out, cut)
            ref = U.best_shift(x, w, cut)
            torch.cuda.synchronize()
            assert torch.equal(out[1], ref[1]) and torch.equal(out[0], ref[0])
    small = mipgen.powerlaw(5, n=900, m=700, nnz=9000, cap=300)
    S, T = chap.Problem(small), chap.Problem(small, row_stage=-1)
    say("scratch limit walks")
    refs = [U.tabu_run(12, 5, 4), T.tabu_run(12, 5, 9)]
    for what, runs in (("single", [G.tabu_run(12, 5, 4), S.tabu_run(12, 5, 9)]),
                       ("batch", chap.batch_run([G, S], [0, 1], [4, 9], 12, 5))):
        for a, b in zip(runs, refs):
            assert np.array_equal(a.trace["var"], b.trace["var"]), what
            assert np.array_equal(a.trace["score"], b.trace["score"]), what
            assert np.array_equal(a.x, b.x) and np.array_equal(a.resid, b.resid), what

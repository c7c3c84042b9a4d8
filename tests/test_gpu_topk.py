"""The proposal set's selection where keys tie, over several compaction chunks
(4096 columns each): a network of equal scores proposes the columns of lowest
internal index, one that scores binary columns 1 and all others 0 proposes the
binary columns first and fills up with the others of lowest internal index; sets
ascend in internal index. A set of at least every column gives that order."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
from oracle import mlp
from test_gpu_parity import chap, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _set(chap, G, flat, K):
    M = chap.Model(0)
    M.set_params(flat.astype(np.float32))
    run = chap.learned_run(G, M, 3, 10, 0, full_every=8, topk=K, train_steps=0, log_sets=1)
    return np.array(run.proposal_set(1))


@pytest.mark.parametrize("n", [255, 4095, 4097, 8192])
def test_ties_over_chunks(chap, n):
    mip = mipgen.random_mixed(n, n=n, m=n // 2, max_row_nnz=8, int_width=30, frac_int=0.7)
    binary = (mip.is_int == 1) & (mip.lb == 0) & (mip.ub == 1)
    flat = np.zeros(mlp.NPARAM)
    G = chap.Problem(mip)
    order = _set(chap, G, flat, 8192)
    assert np.array_equal(np.sort(order), np.arange(n))
    flags = flat.copy()
    flags[4] = flags[1088] = flags[5248] = 1.0   # W1[0][4], W2[0][0], W3[0]: y = the binary input
    nb = int(binary.sum())
    for K in sorted({1, 2, n // 3, max(1, nb - 1), nb + 1, nb + (n - nb) // 2, n - 1}):
        say(f"ties n={n} K={K} binary={nb}")
        assert np.array_equal(_set(chap, G, flat, K), order[:K])
        b = binary[order]
        take = np.zeros(n, dtype=bool)
        take[np.flatnonzero(b)[:K]] = True
        take[np.flatnonzero(~b)[:max(0, K - nb)]] = True
        assert np.array_equal(_set(chap, G, flags, K), order[take])

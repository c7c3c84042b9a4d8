"""The proposal set's selection with more columns than its workgroups have tiles
(4,194,304): every workgroup then compacts two tiles of 4096 columns. Equal keys
and keys above the threshold fall in first and second tiles, the cut among the
equal ones in either."""
from __future__ import annotations

import numpy as np
import pytest

import mipgen
from oracle import mlp
from test_gpu_parity import chap, say  # noqa: F401  (fixture)
from test_gpu_topk import _set

pytestmark = pytest.mark.gpu


def test_two_tiles_a_workgroup(chap):
    n, others, m = 524 * 8192 + 4096 + 1500, 3000, 40
    rng = np.random.default_rng(1)
    wide = np.sort(rng.choice(n, others, replace=False))   # integers in [0, 9], the last columns in internal order
    ub = np.ones(n)
    ub[wide] = 9.0
    rows, cols = np.repeat(np.arange(m), 5), np.sort(rng.choice(wide, 5 * m, replace=False))
    a = mipgen.coo_to_csr_csc(n, m, rows, cols, np.ones(5 * m))
    mip = mipgen.MIP(n=n, m=m, csr_row_ptr=a[0], csr_col=a[1], csr_val=a[2], csc_col_ptr=a[3], csc_row=a[4],
                     csc_val=a[5], sense=np.full(m, ord("G"), dtype=np.uint8), rhs=np.full(m, 3.0), lb=np.zeros(n),
                     ub=ub, is_int=np.ones(n, dtype=np.uint8), obj=np.zeros(n))
    G = chap.Problem(mip, row_stage=-1)
    binary = np.delete(np.arange(n), wide)
    # columns of a lane-group class by degree, then by original index
    deg = np.diff(mip.csc_col_ptr)[wide]
    order = np.concatenate([binary, wide[np.argsort(deg, kind="stable")]])
    flat = np.zeros(mlp.NPARAM)
    up = flat.copy()
    up[5] = up[1088] = up[5248] = 1.0   # W1[0][5], W2[0][0], W3[0]: y = the input "integer and not binary"
    for K in (1, 4095, 4097, 8192):
        say(f"two tiles all equal K={K}")
        assert np.array_equal(_set(chap, G, flat, K), order[:K])
    for K in (1, 1499, 1501, others - 1, others, others + 1, others + 4095, others + 4097, 8192):
        say(f"two tiles K={K}")
        tail = order[n - others:]
        want = np.concatenate([order[:max(0, K - others)], tail[:min(K, others)]])
        assert np.array_equal(_set(chap, G, up, K), want)

"""The autotuner's candidates that plan a problem alike share one time: short_max off
the row-staged form (fractional data, affected rescoring, row_stage = -1), a repeated
candidate, a default written out; candidates whose plans differ are timed each, and
invalid ones stay refused."""
from __future__ import annotations

import pytest

import mipgen
from test_gpu_parity import chap, say  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def test_equal_plans_share_a_time(chap):
    frac = chap.Problem(mipgen.random_mixed(3, n=400, m=300, max_row_nnz=8, integer_data=False))
    whole = chap.Problem(mipgen.powerlaw(3, n=900, m=700, nnz=9000, cap=300))
    say("autotune equal plans")
    best, ms = chap.autotune(frac, walk_iters=64)   # short_max {4, 8} x chunks {2048, 4096} x graphs {32, 64}
    assert list(ms[:4]) == list(ms[4:]) and len(set(ms[:4])) > 1
    assert best.short_max == 8
    _, ms = chap.autotune(whole, walk_iters=64)
    assert any(ms[k] != ms[k + 4] for k in range(4))
    apart = False
    for opts in (dict(row_stage=-1), dict(rescore_cap=32)):
        c = [dict(short_max=s, **opts) for s in (4, 8)] + [dict(short_max=8, chunk_min=4096, **opts),
                                                           dict(short_max=4, chunk_min=2, **opts)]
        _, ms = chap.autotune(whole, c, walk_iters=64)
        assert ms[0] == ms[1] == ms[2], opts
        apart |= ms[3] != ms[0]
    assert apart
    with pytest.raises(chap.ChapError):
        chap.autotune(frac, [dict(short_max=4), dict(short_max=9)], walk_iters=4)

"""The in-transit norms of the value-bounded views, kernel against definition (MI355X).

Every delay count goes through its own form of the reduction (1, 2, 3-4, 5 and more at a time, with
a remainder), tables smaller than a workgroup and larger than one pass of all of them, and the
view that the last workgroup picks must be the stalest whose exported norm fits the bound.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N, M, K, s, bound", [(1, 1, 1, 1, 0.01), (5, 4, 8, 2, 0.02), (300, 100, 33, 3, 0.02),
                                              (3000, 500, 64, 5, 0.02), (700, 90, 20, 8, 0.05), (700, 90, 20, 9, 0.05),
                                              (90, 40, 130, 17, 0.05), (60_000, 9000, 128, 4, 0.01)])
def test_norms_and_views_match_their_definition(N, M, K, s, bound):
    from paper_1410_8043_amd import ps_mf

    print(f"vap norms: N={N} M={M} K={K} s={s}", flush=True)
    rng = np.random.default_rng(N + s)
    nnz = min(N * M, 20 * (N + M))
    cell = rng.choice(N * M, nnz, replace=False)
    user, item = (cell // M).astype(np.int32), (cell % M).astype(np.int32)
    clocks = s + 3
    with ps_mf.PsMf(N, M, K, 3, s, 0.05, 0.01, policy=ps_mf.VAP, value_bound=bound) as g:
        g.load_ratings(user, item, rng.integers(1, 6, nnz).astype(np.float32))
        L, R = (rng.normal(0, 0.1, (n, K)).astype(np.float32) for n in (N, M))
        g.set_factors(L, R)
        hist = [np.concatenate([L.ravel(), R.ravel()])]
        for _ in range(clocks):
            g.clock(1)
            L, R = g.get_factors()
            hist.append(np.concatenate([L.ravel(), R.ravel()]))
        norms = g.export_index(ps_mf.IDX_VAP_NORMS).reshape(clocks, s + 1)
        views = g.export_index(ps_mf.IDX_VERSION_LOG).reshape(clocks, 3)
    for c in range(clocks):
        d = 0
        for k in range(1, min(c, s) + 1):
            want = np.abs(hist[c] - hist[c - k]).max()  # the same fp32 differences: the same bits
            assert norms[c, k] == want, (c, k, norms[c, k], want)
            if float(want) <= bound / np.sqrt(c + 1):
                d = k
        assert (views[c] == c - d).all(), (c, views[c], d)

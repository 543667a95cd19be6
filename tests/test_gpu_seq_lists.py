"""The sequential step by lists (one launch per clock) and by chains (MI355X) against the oracle.

Every case runs in both forms, which must agree bit for bit: lists shorter and longer than a block of
60 records, a user with every item, an item with every user (its row is handed from list to list),
ranks on both sides of each lane width, a row version per client, more workers than users, one
sub-epoch and more than items.  The last case is one worker's long chains, replayed from graphs and
launched one by one.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

TOL = 1e-4  # factors of order 1 after a few clocks in fp32, as in the parity tests


def problem(seed, N, M, nnz, K, hot_user=False, hot_item=False):
    rng = np.random.default_rng(seed)
    cell = rng.choice(N * M, nnz, replace=False)
    user, item = (cell // M).astype(np.int32), (cell % M).astype(np.int32)
    if hot_user:
        user, item = np.r_[user, np.full(M, 3, np.int32)], np.r_[item, np.arange(M, dtype=np.int32)]
    if hot_item:
        user, item = np.r_[user, np.arange(N, dtype=np.int32)], np.r_[item, np.full(N, 2, np.int32)]
    val = rng.integers(1, 6, user.shape[0]).astype(np.float32)
    return user, item, val, rng.normal(0, 0.1, (N, K)).astype(np.float32), rng.normal(0, 0.1, (M, K)).astype(np.float32)


def by_hand(w, N, M, K, P, s, B, G, policy, clocks, lists, graphs=None):
    from paper_1410_8043_amd import ps_mf

    user, item, val, L0, R0 = w
    with ps_mf.PsMf(N, M, K, P, s, 0.01, 0.05, policy=policy, step=ps_mf.STEP_SEQ, B=B, mb_seed=9, strata=G,
                    seq_graphs=graphs, seq_lists=lists) as g:
        g.load_ratings(user, item, val)
        assert all(g.export_index(ps_mf.IDX_SEQ_LISTS, b).size == (16 * P + 1 if lists else 0) for b in range(B))
        g.set_factors(L0, R0)
        g.clock(clocks)
        return g.get_factors()


def by_oracle(w, N, M, K, P, s, B, G, policy, clocks):
    user, item, val, L0, R0 = w
    o = oracle.Oracle(N, M, K, P, s, 0.01, 0.05, policy, oracle.SEQ, B, 9, strata=G)
    o.load(user, item, val)
    o.set_factors(L0, R0)
    o.clock(clocks)
    Lo, Ro = o.get_factors()
    o.close()
    return Lo, Ro


@pytest.mark.parametrize("N, M, nnz, K, P, s, B, G, policy, hot_user, hot_item", [
    (40, 30, 17, 8, 3, 0, 1, 256, oracle.SSP_LAZY, False, False),
    (64, 50, 900, 64, 1, 1, 1, 7, oracle.SSP_LAZY, False, False),
    (200, 70, 3000, 65, 2, 2, 1, 64, oracle.SSP_LAZY, True, False),
    (300, 90, 4000, 33, 2, 1, 1, 16, oracle.ESSP, True, True),
    (300, 90, 4000, 200, 5, 2, 3, 256, oracle.SSP_ROW, False, True),
    (150, 200, 2000, 300, 4, 1, 2, 32, oracle.SSP_WORST, True, True),
    (20, 400, 1500, 128, 37, 3, 1, 256, oracle.ESSP_ROW, True, False),
    (1000, 40, 6000, 16, 4, 2, 1, 1, oracle.SSP_LAZY, False, True),
    (100, 60, 1500, 512, 3, 2, 2, 16, oracle.SSP_ROW, True, True),
    (60, 300, 2500, 20, 64, 1, 1, 1, oracle.ESSP_ROW, True, True),
])
def test_lists_and_chains_match_the_oracle(N, M, nnz, K, P, s, B, G, policy, hot_user, hot_item):
    print(f"lists: N={N} M={M} nnz={nnz} K={K} P={P} s={s} B={B} G={G} policy={policy}", flush=True)
    w = problem(nnz, N, M, nnz, K, hot_user, hot_item)
    args = (w, N, M, K, P, s, B, G, policy, 2 * B + s)
    L, R = by_hand(*args, lists=1)
    Lc, Rc = by_hand(*args, lists=0)
    Lo, Ro = by_oracle(*args)
    assert np.isfinite(Lo).all() and max(np.abs(L - Lo).max(), np.abs(R - Ro).max()) <= TOL
    assert np.array_equal(L, Lc) and np.array_equal(R, Rc)


def test_long_chains_match_the_oracle_with_and_without_graphs():
    N, M, nnz, K, P, G = 4000, 40, 60_000, 20, 1, 8
    print(f"chains: N={N} M={M} nnz={nnz} K={K} P={P} G={G}", flush=True)
    args = (problem(1, N, M, nnz, K), N, M, K, P, 1, 1, G, oracle.SSP_LAZY, 5)
    L, R = by_hand(*args, lists=0, graphs=True)
    Lo, Ro = by_oracle(*args)
    assert np.isfinite(Lo).all() and max(np.abs(L - Lo).max(), np.abs(R - Ro).max()) <= TOL
    Le, Re = by_hand(*args, lists=0, graphs=False)
    assert np.array_equal(L, Le) and np.array_equal(R, Re)


def test_lists_keep_no_second_copy_of_the_ratings_on_the_host():
    """A handle in lists holds as much host memory as one in chains: its records (16 bytes a
    rating, 48 MB here) are freed once they are on the device; 4 bytes a rating of slack."""
    from paper_1410_8043_amd import ps_mf

    def resident():
        with open("/proc/self/statm") as f:
            return int(f.read().split()[1]) * 4096

    N, M, n = 30_000, 1000, 3_000_000
    rng = np.random.default_rng(3)
    user, item = rng.integers(0, N, n).astype(np.int32), rng.integers(0, M, n).astype(np.int32)
    val = np.ones(n, np.float32)
    kept = []
    for lists in (0, 1, 0, 1):  # the first pair warms the allocators up
        g = ps_mf.PsMf(N, M, 8, 64, 0, 0.01, 0.05, step=ps_mf.STEP_SEQ, seq_lists=lists)
        before = resident()
        g.load_ratings(user, item, val)
        kept.append(resident() - before)
        g.close()
    print(f"host bytes kept: {kept}", flush=True)
    assert kept[3] <= kept[2] + 4 * n, kept

"""The commit of items at the edge between few and many partial rows (MI355X).

Up to rank 128, where most items have at most 8 partial rows, those are committed by one thread per 4
columns and the others by a workgroup each; where most have more, and where most have any beyond
rank 128, every item takes a workgroup.  With units of 8 ratings and P workers of one class, an item of n ratings has
ceil(n / 8) partial rows: 0, 1, 3, 4, 5, 8, 9 and 40 of them here (with more classes, up to one
more per class), and 0, 1, 9, 10, 12, 13, 16, 38 and 40 where most have more than 8.  Every
version in the ring against the oracle, factors within 1e-5: rows of
magnitude 1, eta = 0.05, sums of up to 320 products in 32 bits, 320 * 2^-24 = 2e-5 of the step.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

FEW = [0, 1, 8, 20, 32, 33, 64, 65, 320, 0, 7]
MANY = [0, 1, 72, 80, 320, 300, 96, 128, 65, 104, 7]
COLD = [0, 0, 0, 70, 0, 0, 0, 7, 0, 0, 0]


@pytest.mark.parametrize("degrees", [FEW, MANY, COLD], ids=["few", "many", "cold"])
@pytest.mark.parametrize("K", [3, 32, 100, 256, 512])
@pytest.mark.parametrize("s, P, policy", [(0, 3, oracle.SSP_LAZY), (3, 8, oracle.SSP_LAZY), (2, 1, oracle.SSP_LAZY),
                                          (6, 20, oracle.SSP_LAZY), (3, 8, oracle.SSP_ROW), (2, 5, oracle.VAP)])
def test_items_of_few_and_many_partial_rows(K, s, P, policy, degrees):
    from paper_1410_8043_amd import ps_mf

    print(f"commit items: K={K} s={s} P={P} policy={policy} degrees={degrees}", flush=True)
    rng = np.random.default_rng(K + s)
    N, M = 330, len(degrees)
    item = np.repeat(np.arange(M, dtype=np.int32), degrees)
    user = np.concatenate([rng.choice(N, d, replace=False) for d in degrees]).astype(np.int32)
    val = rng.integers(1, 6, item.size).astype(np.float32)
    L0 = (rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32)
    R0 = (rng.standard_normal((M, K)) / np.sqrt(K)).astype(np.float32)
    more = {"value_bound": 0.05} if policy == oracle.VAP else {}
    o = oracle.Oracle(N, M, K, P, s, 0.05, 0.1, policy, oracle.ROWMEAN, 1, 0, None, **more)
    o.load(user, item, val)
    o.set_factors(L0, R0)
    with ps_mf.PsMf(N, M, K, P, s, 0.05, 0.1, policy=policy, unit_max=8, poison=True, **more) as g:
        g.load_ratings(user, item, val)
        g.set_factors(L0, R0)
        for c in range(1, 2 * s + 4):
            g.clock(1)
            o.clock(1)
            L, R = g.get_factors()
            Lo, Ro = o.get_factors()
            assert max(np.abs(L - Lo).max(), np.abs(R - Ro).max()) <= 1e-5, c
    o.close()

"""The LDA sampler's topics per lane and its row accesses, bit for bit against the oracle (MI355X).

Ranks where a lane's topics move by one instruction (two or four a lane, a multiple of that) and
their neighbours where they don't, with few topics in the last lane or none; both addressing
forms; priors far from 1, whose weights span hundreds of binary orders (the smallest floor to 0).
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flat", [False, True])
@pytest.mark.parametrize("K, alpha, beta", [(64, 0.1, 0.01), (66, 0.1, 0.01), (67, 0.1, 0.01), (100, 0.1, 0.01),
                                            (126, 5.0, 1e-9), (128, 1e-60, 1e-60), (192, 0.1, 0.01), (196, 1e-9, 0.5),
                                            (254, 0.1, 0.01), (256, 1e30, 1e-30), (384, 0.1, 0.01), (512, 0.1, 0.01)])
def test_topics_per_lane(K, alpha, beta, flat):
    from paper_1410_8043_amd import ps_lda

    print(f"lda lanes: K={K} alpha={alpha} beta={beta} flat={flat}", flush=True)
    D, V, P, s, B, n = 40, 90, 5, 1, 2, 3000
    rng = np.random.default_rng(K)
    doc = np.sort(rng.integers(0, D, n)).astype(np.int32)
    word, z0 = rng.integers(0, V, n).astype(np.int32), rng.integers(0, K, n).astype(np.int32)
    g = ps_lda.PsLda(D, V, K, P, s, alpha, beta, policy=ps_lda.SSP_LAZY, B=B, seed=K, flat=flat)
    g.load(doc, word, z0)
    o = oracle.LdaOracle(D, V, K, P, s, alpha, beta, 0, B, K)
    o.load(doc, word, z0)
    for _ in range(2):
        g.clock(2)
        o.clock(2)
        assert np.array_equal(g.z(), o.z()) and np.array_equal(g.nwk(), o.nwk()) and np.array_equal(g.ndk(), o.ndk())
    g.close()
    o.close()

"""The LDA commit: version c + every worker's changes, bit for bit against the oracle (MI355X).

Vocabularies on both sides of each words-per-workgroup step and of its last workgroup, worker
counts on both sides of a list's 512, ranks moved by four counts a lane and by one, one and more
loads a row, and words that every worker writes next to words that none does.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V, P, K, n", [(1, 3, 5, 400), (3, 600, 4, 4000), (5, 64, 63, 2000), (8193, 65, 100, 6000),
                                        (16_385, 7, 260, 3000), (32_769, 513, 12, 20_000), (33, 1025, 129, 9000),
                                        (70, 511, 512, 3000), (40, 512, 301, 3000)])
def test_commit_sums_every_workers_changes(V, P, K, n):
    from paper_1410_8043_amd import ps_lda

    print(f"lda commit: V={V} P={P} K={K} tokens={n}", flush=True)
    D = P + 5
    rng = np.random.default_rng(V + P)
    doc = np.sort(rng.integers(0, D, n)).astype(np.int32)
    # half of the tokens on few words, so that most workers write them
    word = np.where(rng.random(n) < 0.5, rng.integers(0, min(V, 3), n), rng.integers(0, V, n)).astype(np.int32)
    z0 = rng.integers(0, K, n).astype(np.int32)
    g = ps_lda.PsLda(D, V, K, P, 1, 0.1, 0.01, policy=ps_lda.SSP_LAZY, B=2, seed=3)
    g.load(doc, word, z0)
    o = oracle.LdaOracle(D, V, K, P, 1, 0.1, 0.01, 0, 2, 3)
    o.load(doc, word, z0)
    for _ in range(3):
        g.clock(1)
        o.clock(1)
        assert np.array_equal(g.nwk(), o.nwk())
    assert np.array_equal(g.z(), o.z())
    g.close()
    o.close()

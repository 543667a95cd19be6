"""Factors and assignments cross to the host unchanged (MI355X).

Ranks equal to their padded rank move in one contiguous copy; the others through a pack
buffer of 16 MiB, in pieces.  The rows must come back bit for bit at ranks on both sides of
a power of two and of a wavefront, and where the table needs one piece, exactly one, and a
last piece of one row; the padding columns must stay zero (a clock's products read them).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

PIECE = 16 << 20


@pytest.mark.parametrize("K, users", [(1, 5), (7, 33), (8, 100), (63, 65), (64, 65), (65, 65), (100, 1),
                                      (100, PIECE // 400), (100, PIECE // 400 + 1), (129, 3 * (PIECE // 516) - 1),
                                      (511, 17)])
def test_factors_come_back_bit_for_bit(K, users):
    from paper_1410_8043_amd import ps_mf

    print(f"transfers: K={K} users={users}", flush=True)
    items = 3
    rng = np.random.default_rng(K)
    L0 = rng.standard_normal((users, K), dtype=np.float32)
    R0 = rng.standard_normal((items, K), dtype=np.float32)
    with ps_mf.PsMf(users, items, K, 1, 1, 0.0, 0.0) as g:
        g.load_ratings([users - 1], [1], [2.0])
        for _ in range(2):
            g.set_factors(L0, R0)
            L, R = g.get_factors()
            assert np.array_equal(L, L0) and np.array_equal(R, R0)
            # padding columns are zero: the one rating's loss is that of the K columns alone
            want = (2.0 - float(L0[-1].astype(np.float64) @ R0[1].astype(np.float64))) ** 2
            assert abs(g.loss() - want) <= 1e-5 * max(1.0, want)
            g.clock(2)  # eta = 0: every version equals the first
            L, R = g.get_version(1)
            assert np.array_equal(L, L0) and np.array_equal(R, R0)
            L0, R0 = L0[::-1].copy(), -R0


@pytest.mark.parametrize("tokens, D, P, B", [(1, 1, 1, 1), (255, 9, 3, 2), (257, 300, 4, 3), (4099, 50, 7, 2)])
def test_assignments_come_back_in_load_order(tokens, D, P, B):
    from paper_1410_8043_amd import ps_lda

    print(f"transfers: tokens={tokens} D={D} P={P} B={B}", flush=True)
    rng = np.random.default_rng(tokens)
    doc, word, z0 = (rng.integers(0, n, tokens).astype(np.int32) for n in (D, 11, 70))
    g = ps_lda.PsLda(D, 11, 70, P, 1, 0.1, 0.01, B=B, seed=5)
    g.load(doc, word, z0)
    assert np.array_equal(g.z(), z0)
    g.clock(2)
    z = g.z()
    ndk = np.zeros((D, 70), np.int32)
    np.add.at(ndk, (doc, z), 1)
    assert np.array_equal(ndk, g.ndk())
    g.close()

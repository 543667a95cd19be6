"""The squared loss at the edges of its segments (MI355X).

A lane group sweeps up to 64 ratings of one user (from rank 129 on, up to 95 where they are all, else 48
to 80), 8 pairs at a time, read 8 ahead from any 4-byte address.  Users of 1, 7, 8, 9, 63, 64, 65, 95,
96, 127, 129, 159, 160, 511, 512 and 513 ratings follow one another here, so segments start at
every remainder of 8, and the last one ends the arrays.  Where the segments are more than the
static scratch has partial sums, each lane group sweeps several: the last test.
The sum must be that of the same residuals in 64 bits: a residual holds K products summed in
32 bits, whose relative error is at most (K + 1) 2^-24 of the products' magnitudes, at most
2^-24 * 513 * 2 of the squares' sum at these values; 1e-5 allows a sixth of that.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DEGREES = [1, 7, 8, 9, 63, 64, 65, 95, 96, 127, 129, 159, 160, 511, 512, 513]


@pytest.mark.parametrize("K", [1, 8, 16, 33, 64, 100, 128, 256, 512])
@pytest.mark.parametrize("B, last", [(1, 1), (3, 5)])
def test_loss_of_users_at_segment_edges(K, B, last):
    from paper_1410_8043_amd import ps_mf

    print(f"loss segments: K={K} B={B} last={last}", flush=True)
    rng = np.random.default_rng(K)
    degrees = [0, *DEGREES, 0, last]
    M, N = 600, len(degrees)
    user = np.repeat(np.arange(N), degrees)
    item = np.concatenate([rng.choice(M, d, replace=False) for d in degrees]).astype(np.int32)
    val = rng.standard_normal(user.size).astype(np.float32)
    L = (rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32)
    R = rng.standard_normal((M, K)).astype(np.float32)
    with ps_mf.PsMf(N, M, K, 2, 1, 0.0, 0.0, B=B, mb_seed=7) as g:
        g.load_ratings(user, item, val)
        g.set_factors(L, R)
        got, static = g.loss(), ps_mf.ps_mf_loss_noalloc(g.h)
    e = val.astype(np.float64) - (L[user].astype(np.float64) * R[item].astype(np.float64)).sum(1)
    want = float((e * e).sum())
    assert got == static
    assert abs(got - want) <= 1e-5 * want, (got, want)


def test_loss_where_a_lane_group_sweeps_several_segments():
    """2^18 workgroups of 32 lane groups (rank 32) hold 8.4M segments: with that many users of one
    rating and 2000 of 600, the launch takes the workgroups of segments of 512, and the last
    16,000 segments are swept in a second turn.  The static scratch cannot hold as many."""
    from paper_1410_8043_amd import ps_mf

    many, busy, d, K, M = (1 << 18) * 32 + 100, 2000, 600, 17, 700
    print(f"loss segments: {many} users of 1, {busy} of {d} ratings, K={K}", flush=True)
    rng = np.random.default_rng(11)
    user = np.concatenate([np.arange(many), np.repeat(np.arange(many, many + busy), d)]).astype(np.int32)
    item = np.concatenate([rng.integers(0, M, many), (np.arange(busy * d) * 7) % M]).astype(np.int32)
    val = rng.standard_normal(user.size, dtype=np.float32)
    L = rng.standard_normal((many + busy, K), dtype=np.float32)
    R = rng.standard_normal((M, K), dtype=np.float32) / 4
    with ps_mf.PsMf(many + busy, M, K, 2, 0, 0.0, 0.0) as g:
        g.load_ratings(user, item, val)
        g.set_factors(L, R)
        got = g.loss()
        assert got == g.loss()
        with pytest.raises(ps_mf.PsMfError) as e:
            ps_mf.ps_mf_loss_noalloc(g.h)
        assert e.value.code == ps_mf.EINVAL
    want = 0.0
    for a in range(0, user.size, 1 << 20):
        u, i = user[a:a + (1 << 20)], item[a:a + (1 << 20)]
        e = val[a:a + (1 << 20)].astype(np.float64) - (L[u].astype(np.float64) * R[i].astype(np.float64)).sum(1)
        want += float((e * e).sum())
    assert abs(got - want) <= 1e-5 * want, (got, want)

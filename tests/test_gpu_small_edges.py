"""The one-launch Beaver matmul at the edges of its two kernels (k lanes of 16 and of 128, 4 x 4 blocks of outputs) and
of the range in which a short k takes it, against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import dev, pair, say

pytestmark = pytest.mark.gpu

SEED, DSEED = 2071, 3071


@pytest.fixture(scope="module")
def m():
    import paper_2109_00984_amd as mpc
    return mpc


@pytest.fixture(scope="module")
def c(m):
    ctx = m.Context(device=0, seed=SEED)
    yield ctx
    ctx.close()


@pytest.mark.parametrize("M,N,K", [(1, 1, 0), (1, 1, 1), (5, 7, 1), (4, 4, 15), (3, 5, 16), (9, 6, 17), (33, 30, 111), (21, 34, 112), (33, 30, 126), (64, 48, 127), (61, 47, 128),
                                   (17, 19, 129), (5, 3, 255), (6, 9, 256), (7, 2, 257), (512, 511, 1), (513, 512, 1), (300, 700, 3), (1, 9000, 17),
                                   (9001, 1, 16), (16, 4099, 5), (1, 2000, 49), (2, 3, 1023), (3, 2, 1024)])
@pytest.mark.parametrize("form", ["auto", "plain"])
def test_matches_oracle(m, c, M, N, K, form):
    say(f"small Beaver matmul {M}x{N}x{K} {form}")
    tag = M + 7 * N + 11 * K
    g = np.random.default_rng(tag)
    X, Y = (g.integers(0, 2**64, size=s, dtype=np.uint64) for s in ((M, K), (K, N)))
    x, y = c.share(dev(X), 0, 1), c.share(dev(Y), 1, 2)
    t = c.dealer(m.TRIPLE_MATMUL, DSEED, tag, (M, N, K))
    got = pair(c, c.beaver_matmul(x, y, t, 16, form))
    want = oracle.beaver_matmul(oracle.share(X, 0, SEED, 1), oracle.share(Y, 1, SEED, 2), oracle.dealer_matmul(DSEED, tag, M, N, K), 16)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])


@pytest.mark.parametrize("M,N,K", [(2048, 2050, 8), (2048, 2050, 9), (96, 43691, 8), (95, 23000, 1), (16, 30000, 15)])
def test_short_k_forms_agree(m, c, M, N, K):
    """What AUTO takes for k below 16 against the plain form, for every call that chooses."""
    say(f"short k {M}x{N}x{K}")
    g = np.random.default_rng(M + K)
    A, B = (dev(g.integers(0, 2**64, size=s, dtype=np.uint64)) for s in ((M, K), (K, N)))
    want = c.ring_gemm(A, B, "plain")
    assert (c.ring_gemm(A, B) == want).all()
    t = c.dealer(m.TRIPLE_MATMUL, DSEED, 5, (M, N, K))
    assert (t.c0 + t.c1 == c.ring_gemm(t.a0 + t.a1, t.b0 + t.b1, "plain")).all()
    x, y = c.share(A, 0, 1), c.share(B, 1, 2)
    z, p = c.beaver_matmul(x, y, t, 16), c.beaver_matmul(x, y, t, 16, "plain")
    assert (z.s0 == p.s0).all() and (z.s1 == p.s1).all()
    xs, ys, tm = c.mp_share(A, 3, 0, 1), c.mp_share(B, 3, 1, 2), c.mp_dealer(3, m.TRIPLE_MATMUL, DSEED, 6, (M, N, K))
    assert (c.mp_reveal(c.mp_beaver_matmul(xs, ys, tm)) == want).all()


@pytest.mark.parametrize("P", [8, 9, 16])
@pytest.mark.parametrize("M,N,K", [(1, 1, 0), (1, 1, 1), (37, 5, 65), (64, 96, 128), (33, 300, 70), (512, 480, 260), (513, 490, 260)])
def test_many_parties(m, c, P, M, N, K):
    """The limb form's fused open and pack, and a pack job per party where the parties are many and the blocks few."""
    say(f"{P} parties {M}x{N}x{K}")
    g = np.random.default_rng(P + K)
    X, Y = (g.integers(0, 2**64, size=s, dtype=np.uint64) for s in ((M, K), (K, N)))
    x, y = c.mp_share(dev(X), P, 0, 1), c.mp_share(dev(Y), P, P - 1, 2)
    t = c.mp_dealer(P, m.TRIPLE_MATMUL, DSEED, 7, (M, N, K))
    want = oracle.ring_gemm(X, Y)
    p = c.mp_beaver_matmul(x, y, t, "plain")
    for form in ("limb8", "auto"):
        z = c.mp_beaver_matmul(x, y, t, form)
        assert np.array_equal(c.mp_reveal(z).cpu().numpy().view(np.uint64), want)
        assert all((a == b).all() for a, b in zip(z, p))

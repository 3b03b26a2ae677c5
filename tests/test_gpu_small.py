"""Small products: the one-launch Beaver matmul at the edges of its range and of its 4x4 tiles and 32 lanes of k, the
limb form on products of a few tiles (k slices whose tables travel in the kernel arguments), and AUTO without a
workspace."""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import dev, host, pair, say

pytestmark = pytest.mark.gpu

SEED, DSEED = 2061, 3061


@pytest.fixture(scope="module")
def m():
    import paper_2109_00984_amd as mpc
    return mpc


@pytest.fixture(scope="module")
def c(m):
    ctx = m.Context(device=0, seed=SEED)
    yield ctx
    ctx.close()


def rnd(seed, shape):
    return np.random.default_rng(seed).integers(0, 2**64, size=shape, dtype=np.uint64)


@pytest.mark.parametrize("M,N,K,launches", [(1, 1, 1, 1), (4, 4, 32, 1), (5, 3, 33, 1), (3, 7, 31, 1), (64, 48, 1024, 1), (128, 10, 1024, 1),
                                            (1024, 3, 1023, 1), (128, 128, 128, 1), (1, 3072, 1024, None), (1, 1536, 1024, 1), (1, 1540, 1024, None), (65, 48, 1024, None),
                                            (16, 24, 1025, None), (7, 9, 2049, None)])
@pytest.mark.parametrize("trunc", [0, 16])
def test_beaver_matmul_auto(m, c, M, N, K, launches, trunc):
    say(f"small Beaver matmul {M}x{N}x{K} trunc {trunc}")
    tag = M + 7 * N + 11 * K
    X, Y = rnd(tag, (M, K)), rnd(tag + 1, (K, N))
    x, y = c.share(dev(X), 0, 1), c.share(dev(Y), 1, 2)
    t = c.dealer(m.TRIPLE_MATMUL, DSEED, tag, (M, N, K))
    before = c.stats()["launches"]
    z = c.beaver_matmul(x, y, t, trunc)
    if launches is not None:
        assert c.stats()["launches"] - before == launches
    ot = oracle.dealer_matmul(DSEED, tag, M, N, K)
    want = oracle.beaver_matmul(oracle.share(X, 0, SEED, 1), oracle.share(Y, 1, SEED, 2), ot, trunc)
    got = pair(c, z)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    assert np.array_equal(host(c, t.c1), ot.c[1])


@pytest.mark.parametrize("M,N,K", [(1, 1, 15), (1, 1, 16), (16, 16, 256), (4, 4, 8192), (200, 100, 50), (33, 129, 700), (70, 20, 4100),
                                   (1, 1000, 1000), (130, 1, 40000)])
def test_ring_gemm_auto(c, M, N, K):
    say(f"small ring GEMM {M}x{N}x{K}")
    A, B = rnd(M + K, (M, K)), rnd(N + K + 1, (K, N))
    want = oracle.ring_gemm(A, B)
    for form in ("auto", "limb8", "plain"):
        assert np.array_equal(host(c, c.ring_gemm(dev(A), dev(B), form)), want), form


@pytest.mark.parametrize("M,N,K", [(81, 3157, 1000), (512, 1024, 1100), (500, 1100, 130), (777, 1500, 1001), (1500, 1000, 1030),
                                   (1024, 1537, 777), (300, 200, 20000)])
def test_k_slices(m, c, M, N, K):
    """The limb form where its tiles leave a round of the chip partly empty (k slices), up to past the last size that
    is sliced, eager and replayed, against the plain form."""
    say(f"k slices {M}x{N}x{K}")
    x, y = c.share(dev(rnd(M, (M, K))), 0, 1), c.share(dev(rnd(N, (K, N))), 1, 2)
    t = c.dealer(m.TRIPLE_MATMUL, DSEED, K, (M, N, K))
    want = c.beaver_matmul(x, y, t, 16, "plain")
    z = c.beaver_matmul(x, y, t, 16, "limb8")
    c.sync()
    assert torch.equal(z.s0, want.s0) and torch.equal(z.s1, want.s1)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        g = m.Context(device=0, seed=SEED)
        g.beaver_matmul(x, y, t, 16, "limb8", out=z)
        g.sync()
        g.graph_begin()
        g.beaver_matmul(x, y, t, 16, "limb8", out=z)
        gr = g.graph_end()
        for _ in range(2):
            z.s0.zero_()
            z.s1.zero_()
            g.graph_launch(gr)
            g.sync()
            assert torch.equal(z.s0, want.s0) and torch.equal(z.s1, want.s1)
        m.Context.graph_destroy(gr)
        g.close()


@pytest.mark.parametrize("P", [2, 3, 7])
@pytest.mark.parametrize("M,N,K", [(5, 9, 17), (64, 32, 128), (20, 300, 2000)])
def test_party_matmul_auto(m, c, P, M, N, K):
    X, Y = rnd(1, (M, K)), rnd(2, (K, N))
    x, y = c.mp_share(dev(X), P, 0, 1), c.mp_share(dev(Y), P, 1, 2)
    t = c.mp_dealer(P, m.TRIPLE_MATMUL, DSEED, 4, (M, N, K))
    z = c.mp_beaver_matmul(x, y, t)
    assert np.array_equal(host(c, c.mp_reveal(z)), oracle.ring_gemm(X, Y))


def test_auto_without_workspace(m):
    """Under capture a context that has no workspace yet still takes a small product: AUTO falls back."""
    streams = (torch.cuda.Stream(), torch.cuda.Stream())
    c = m.Context(device=0, seed=SEED, streams=streams)
    A, B = rnd(1, (90, 300)), rnd(2, (300, 70))
    with torch.cuda.stream(streams[0]):
        a, b, out = dev(A), dev(B), torch.empty((90, 70), dtype=torch.int64, device="cuda")
        c.sync()
        c.graph_begin()
        c.ring_gemm(a, b, out=out)
        g = c.graph_end()
        for _ in range(2):
            out.zero_()
            c.graph_launch(g)
            c.sync()
            assert np.array_equal(out.cpu().numpy().view(np.uint64), oracle.ring_gemm(A, B))
    c.close()


class _Sub(torch.Tensor):
    pass


def test_native_calls_match_python(m, c, monkeypatch):
    """The native call of every entry point it has, with and without given outputs, equals the Python code's call (which
    runs when the native one answers None, as for a tensor subclass), and what that refuses stays refused."""
    M, N, K = 37, 21, 50
    X, Y = dev(rnd(1, (M, K))), dev(rnd(2, (K, N)))
    t, tm = c.dealer(m.TRIPLE_MATMUL, DSEED, 1, (M, N, K)), c.dealer(m.TRIPLE_MUL, DSEED, 2, (M * K,))
    sq = c.dealer(m.TRIPLE_SQUARE, DSEED, 3, (M * K,))

    def calls(out):
        new = lambda *s: m.SharedPair(c.empty(s), c.empty(s)) if out else None  # noqa: E731
        x, y = c.share(X, 0, 2**63 + 5, out=new(M, K)), c.share(Y, 1, 2, out=new(K, N))
        w = c.share(X, 1, 9)
        z = [c.beaver_matmul(x, y, t, 16, f, out=new(M, N)) for f in ("auto", "plain", "limb8")]
        z += [c.beaver_mul(x, w, tm, 16, out=new(M, K)), c.beaver_mul(x, None, sq, 0, out=new(M, K)), c.beaver_mul(x, None, tm, 3)]
        return [x.s0, x.s1] + [s for p in z for s in p] + [c.reveal(p, out=c.empty(p.shape) if out else None) for p in z]

    native = [calls(False), calls(True)]

    class Off:
        def __getattr__(self, name):
            return lambda *a: None
    with monkeypatch.context() as mp:
        mp.setattr(m, "_binding", Off())
        want = calls(False)
    for got in native:
        assert all(torch.equal(g, w) and g.shape == w.shape for g, w in zip(got, want))
    x, y = c.share(X, 0, 1), c.share(Y, 1, 2)
    ref = c.beaver_matmul(x, y, t, 16)
    sub = m.SharedPair(x.s0.as_subclass(_Sub), x.s1)
    z = c.beaver_matmul(sub, y, t, 16)
    assert torch.equal(z.s0, ref.s0) and torch.equal(z.s1, ref.s1)
    bad = [lambda: c.beaver_matmul(m.SharedPair(x.s0.t(), x.s1.t()), y, t), lambda: c.beaver_matmul(y, x, t),
           lambda: c.beaver_matmul(m.SharedPair(x.s0.to(torch.int32), x.s1), y, t), lambda: c.beaver_matmul(x, y, c.dealer(m.TRIPLE_MUL, DSEED, 4, (700,))),
           lambda: c.beaver_matmul(m.SharedPair(x.s0[:-1], x.s1), y, t), lambda: c.beaver_matmul(m.SharedPair(x.s0.cpu(), x.s1), y, t),
           lambda: c.beaver_mul(x, y, tm), lambda: c.beaver_mul(x, x, sq), lambda: c.reveal(m.SharedPair(x.s0, y.s0)),
           lambda: c.share(X.to(torch.float64), 0, 1), lambda: c.share(X, 0, 1, out=y),
           lambda: c.beaver_matmul(x, y, t, out=m.SharedPair(c.empty((M, N + 1)), c.empty((M, N))))]
    for f in bad:
        with pytest.raises(ValueError):
            f()
    with pytest.raises(m.MPCError):
        c.beaver_matmul(x, y, t, 64)
    with pytest.raises(m.MPCError):
        c.share(X, 2, 1)

"""Residue-form products that plan to each of its tile shapes, and the convolutions' strides, chunks of k and dealt
im2col operands, against the plain form and the oracle.  (That the shapes take the form and the tiles named here is
checked without a GPU in test_host_plan.py; here the launches are counted: one pack, one GEMM per tile shape, one
combine.)"""
import numpy as np
import pytest
import torch

import oracle
from tests.gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

SEED, DSEED = 2081, 3081

MATMULS = [((2751, 330, 3540), [(256, 128), (128, 128)]), ((2830, 361, 3852), [(256, 256), (256, 128)]), ((345, 2836, 3697), [(256, 256), (128, 256)]),
           ((364, 2811, 3262), [(128, 256), (128, 128)]), ((2700, 333, 6007), [(256, 256), (256, 128)]), ((333, 2700, 11003), [(256, 256), (128, 256)])]
# batch, channels in, length, channels out, taps, stride; tiles; chunks of k, and whether one starts inside a tap run
CONVS = [((6, 245, 363, 209, 19, 3), [(128, 128)], 1, False), ((6, 250, 339, 277, 11, 2), [(128, 256)], 1, False),
         ((3, 187, 557, 326, 14, 2), [(256, 128)], 1, False), ((5, 296, 306, 155, 39, 3), [(256, 256)], 3, True),
         ((2, 523, 763, 146, 39, 2), [(256, 256), (128, 128)], 5, True),
         ((4, 141, 2072, 331, 19, 3), [(128, 256), (128, 128)], None, None)]  # with im2col
# the same; whether the dealer packs it without im2col
DEALT = [((3, 125, 1246, 329, 18, 2), [(128, 256)], True), ((6, 113, 402, 523, 38, 2), [(256, 128)], True),
         ((2, 87, 1430, 710, 30, 1), [(256, 256), (128, 128)], False)]


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
    return dev(np.random.default_rng(seed).integers(0, 2**64, size=shape, dtype=np.uint64))


def launches(c, f):
    before = c.stats()["launches"]
    out = f()
    return out, c.stats()["launches"] - before


def check_conv(c, t, s, B, cout, lout):
    """The dealt c at corners and the middle of every axis."""
    a, b = host(c, t.a0 + t.a1), host(c, t.b0 + t.b1)
    at = [np.array([0, n - 1, n // 2]) for n in (B, cout, lout)]
    assert np.array_equal(host(c, t.c0 + t.c1)[tuple(at)], oracle.conv1d_at(a, b, s, *at))


@pytest.mark.parametrize("shape,tiles", MATMULS)
def test_matmul(m, c, shape, tiles):
    M, N, K = shape
    say(f"residue Beaver matmul {M}x{N}x{K} {tiles}")
    x, y = c.share(rnd(M, (M, K)), 0, 1), c.share(rnd(N, (K, N)), 1, 2)
    t = c.dealer(m.TRIPLE_MATMUL, DSEED, 3, shape)
    z, n = launches(c, lambda: c.beaver_matmul(x, y, t, 16))
    assert n == 2 + len(tiles)
    p = c.beaver_matmul(x, y, t, 16, "plain")
    assert torch.equal(z.s0, p.s0) and torch.equal(z.s1, p.s1)


@pytest.mark.parametrize("shape,tiles", [(s, t) for s, t, *_ in CONVS])
def test_conv(m, c, shape, tiles):
    B, cin, L, cout, k, s = shape
    say(f"residue conv {shape} {tiles}")
    x, w = c.share(rnd(1, (B, cin, L)), 0, 1), c.share(rnd(2, (cout, cin, k)), 1, 2)
    t = c.dealer(m.TRIPLE_CONV1D, DSEED, 9, shape)
    z, n = launches(c, lambda: c.beaver_conv1d(x, w, t, s, 16))
    assert n == 2 + len(tiles)
    p = c.beaver_conv1d(x, w, t, s, 16, "plain")
    assert torch.equal(z.s0, p.s0) and torch.equal(z.s1, p.s1)
    check_conv(c, t, s, B, cout, (L - k) // s + 1)


@pytest.mark.parametrize("shape,tiles", [(s, t) for s, t, _ in DEALT])
def test_dealt_conv(m, c, shape, tiles):
    B, cin, L, cout, k, s = shape
    say(f"dealt conv {shape} {tiles}")
    t, n = launches(c, lambda: c.dealer(m.TRIPLE_CONV1D, DSEED, 11, shape))
    assert n == 2 + len(tiles) + 3  # and the fills of the activation's shares and c_0
    check_conv(c, t, s, B, cout, (L - k) // s + 1)
    # against the plain form: the product of the dealt values, with a zero triple
    zero = m.TripleShares(*(torch.zeros_like(v) for v in (t.a0, t.a1, t.b0, t.b1, t.c0, t.c1)))
    z = c.beaver_conv1d(m.SharedPair(t.a0, t.a1), m.SharedPair(t.b0, t.b1), zero, s, 0, "plain")
    assert torch.equal(t.c0 + t.c1, z.s0 + z.s1)

"""Timed cases of the framework: secret-shared products as a private-inference program issues them.

A case is one call, one layer or one short chain of calls of the public Python binding, from the 64x128 @ 128x32
product of a few microseconds to the 4096^3 product and the 256-problem batch.  Every output is a ring element
(int64), so two correct implementations agree bit for bit.
"""
import math
import random

import torch

import paper_2109_00984_amd as mpc

FRAC = 16
SEED, DSEED = 2000, 3000  # the parties' and the dealer's PRG seeds
_ctx = {}


def _context():
    """The program's one context (its workspace stays from call to call)."""
    if "main" not in _ctx:
        _ctx["main"] = mpc.Context(device=0, seed=SEED)
    return _ctx["main"]


# ---------------------------------------------------------------- the cases
# Layer shapes of the 784-1024-1024-10 perceptron, and (Cin, Cout, kernel, stride) of the speech convolution stack
# with the input length of each layer at 1600 samples.
MLP = (784, 1024, 1024, 10)
CONV = [(40, 250, 48, 2, 1600)] + [(250, 250, 7, 1, 777 - 6 * i) for i in range(7)] + [(250, 2000, 32, 1, 735),
                                                                                      (2000, 40, 1, 1, 704)]


def listed():
    return [
        # one small layer of a latency-bound service: launches and host time count
        dict(name="small_matmul", kind="matmul", M=64, N=32, K=128),
        # the element-wise product of a large activation (and its truncation)
        dict(name="mul_2e24", kind="mul", n=1 << 24, square=False),
        # a whole private inference over a perceptron: share the input, three matrix layers, square activations, reveal
        dict(name="mlp_128", kind="mlp", batch=128),
        # a matrix layer whose sizes are no multiples of anything
        dict(name="matmul_ragged", kind="matmul", M=777, N=1500, K=3001),
        # the largest matrix layer: the headline product
        dict(name="matmul_4096", kind="matmul", M=4096, N=4096, K=4096),
        # the online phase over triples that the dealer packed beforehand: share, product, reveal
        dict(name="prepacked_2048", kind="prepacked", M=2048, N=2048, K=2048),
        # the offline phase: the dealer draws a matrix triple
        dict(name="deal_2048", kind="deal", M=2048, N=2048, K=2048),
        # a middle layer of the speech stack, and its largest
        dict(name="conv_250", kind="conv", batch=8, layer=1),
        dict(name="conv_2000", kind="conv", batch=8, layer=8),
        # many uneven products as one call, replayed from a graph as a serving program does
        dict(name="grouped_256", kind="grouped", count=256, shapes=1005, graph=True),
        # a comparison-based activation: A2B, sign bit to arithmetic, product
        dict(name="relu_2e20", kind="relu", n=1 << 20),
        # a matrix layer among three parties with Algorithm 1's truncation
        dict(name="party3_layer", kind="party", P=3, M=512, N=1024, K=1024),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["matmul", "matmul", "mul", "mlp", "prepacked", "deal", "conv", "grouped", "relu", "party"])
    if kind in ("matmul", "prepacked", "deal"):
        top = 4096 if kind == "matmul" else 2048
        return dict(kind=kind, M=_log(rng, 16, top), N=_log(rng, 16, top), K=_log(rng, 32, top))
    if kind == "mul":
        return dict(kind=kind, n=_log(rng, 1 << 10, 1 << 24), square=rng.random() < 0.4)
    if kind == "mlp":
        return dict(kind=kind, batch=_log(rng, 1, 256))
    if kind == "conv":
        return dict(kind=kind, batch=_log(rng, 1, 8), layer=rng.randrange(len(CONV)))
    if kind == "grouped":
        return dict(kind=kind, count=_log(rng, 4, 128), shapes=rng.randrange(1 << 20), graph=rng.random() < 0.5)
    if kind == "relu":
        return dict(kind=kind, n=_log(rng, 1 << 10, 1 << 20))
    return dict(kind=kind, P=rng.choice([2, 3, 4, 5]), M=_log(rng, 16, 512), N=_log(rng, 16, 1024),
                K=_log(rng, 32, 1024))


def _group_shapes(case):
    rng = random.Random(case["shapes"])
    return [(_log(rng, 16, 2048), _log(rng, 16, 1024), _log(rng, 32, 4096)) for _ in range(case["count"])]


# ---------------------------------------------------------------- inputs
class _Inputs:
    """Fixed-point tensors from one seed, uniform as the workloads draw them, and the tags of one case's shares."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        self.tag = 1000 * (seed % 1000003)

    def real(self, shape, scale=4.0):
        x = torch.rand(shape, generator=self.g, device="cuda", dtype=torch.float64)
        return ((x * 2 - 1) * scale * (1 << FRAC)).round().to(torch.int64)

    def next_tag(self):
        self.tag += 1
        return self.tag


def _product(c, d, M, N, K):
    x = c.share(d.real((M, K)), 0, d.next_tag())
    y = c.share(d.real((K, N)), 1, d.next_tag())
    return x, y


def prepare(case, seed):
    d, kind = _Inputs(seed), case["kind"]
    if kind == "grouped":
        # capture needs a stream of its own, so this program binds its context to one
        streams = (torch.cuda.Stream(), torch.cuda.Stream())
        c = mpc.Context(device=0, seed=SEED, streams=streams)
        torch.cuda.synchronize()
        with torch.cuda.stream(streams[0]):
            probs, sizes = [], []
            for M, N, K in _group_shapes(case):
                x, y = _product(c, d, M, N, K)
                probs.append((x, y, c.dealer(mpc.TRIPLE_MATMUL, DSEED, d.next_tag(), (M, N, K))))
                sizes.append((M, N))
            # one buffer per party holds all outputs
            flat = [torch.empty(sum(M * N for M, N in sizes), dtype=torch.int64, device="cuda") for _ in range(2)]
            outs, at = [], 0
            for M, N in sizes:
                outs.append(mpc.SharedPair(*(f[at:at + M * N].view(M, N) for f in flat)))
                at += M * N
            s = dict(kind=kind, c=c, probs=probs, outs=outs, flat=flat, graph=None)
            if case["graph"]:
                c.beaver_matmul_grouped(probs, FRAC, outs=outs)
                c.sync()
                c.graph_begin()
                c.beaver_matmul_grouped(probs, FRAC, outs=outs)
                s["graph"] = c.graph_end()
        torch.cuda.synchronize()
        return s
    c = _context()
    s = dict(kind=kind, c=c)
    if kind in ("matmul", "deal", "prepacked"):
        M, N, K = case["M"], case["N"], case["K"]
        if kind == "deal":
            s.update(tag=d.next_tag(), dims=(M, N, K))
        elif kind == "matmul":
            s["x"], s["y"] = _product(c, d, M, N, K)
            s["t"] = c.dealer(mpc.TRIPLE_MATMUL, DSEED, d.next_tag(), (M, N, K))
        else:
            s.update(x=d.real((M, K)), tag=d.next_tag(), y=c.share(d.real((K, N)), 1, d.next_tag()))
            s["t"], s["packed"] = c.dealer_packed(DSEED, d.next_tag(), (M, N, K))
    elif kind == "mul":
        n, sq = case["n"], case["square"]
        s["x"] = c.share(d.real((n,)), 0, d.next_tag())
        s["y"] = None if sq else c.share(d.real((n,)), 1, d.next_tag())
        s["t"] = c.dealer(mpc.TRIPLE_SQUARE if sq else mpc.TRIPLE_MUL, DSEED, d.next_tag(), (n,))
    elif kind == "mlp":
        B = case["batch"]
        s.update(x=d.real((B, MLP[0]), 1.0), tag=d.next_tag(), layers=[])
        for i, (K, N) in enumerate(zip(MLP, MLP[1:])):
            w = c.share(d.real((K, N), 1.0 / math.sqrt(K)), 1, d.next_tag())
            t = c.dealer(mpc.TRIPLE_MATMUL, DSEED, d.next_tag(), (B, N, K))
            sq = c.dealer(mpc.TRIPLE_SQUARE, DSEED, d.next_tag(), (B * N,)) if i + 2 < len(MLP) else None
            s["layers"].append((w, t, sq))
    elif kind == "conv":
        cin, cout, k, stride, L = CONV[case["layer"]]
        B = case["batch"]
        s["x"] = c.share(d.real((B, cin, L), 2.0), 0, d.next_tag())
        s["w"] = c.share(d.real((cout, cin, k), 1.0 / math.sqrt(cin * k)), 1, d.next_tag())
        s["stride"] = stride
        s["t"] = c.dealer(mpc.TRIPLE_CONV1D, DSEED, d.next_tag(), (B, cin, L, cout, k, stride))
    elif kind == "relu":
        n = case["n"]
        s["x"] = c.share(d.real((n,)), 0, d.next_tag())
        s["tag"] = d.next_tag()
        s["t"] = c.dealer_and(DSEED, d.next_tag(), c.A2B_TRIPLES * n)
        s["rb"], s["ra"] = c.dealer_b2a(DSEED, d.next_tag(), n)
        s["m"] = c.dealer(mpc.TRIPLE_MUL, DSEED, d.next_tag(), (n,))
    else:
        P, M, N, K = case["P"], case["M"], case["N"], case["K"]
        s["x"] = c.mp_share(d.real((M, K)), P, 0, d.next_tag())
        s["y"] = c.mp_share(d.real((K, N)), P, 1, d.next_tag())
        s["t"] = c.mp_dealer(P, mpc.TRIPLE_MATMUL, DSEED, d.next_tag(), (M, N, K))
        s["r"], s["theta"] = c.mp_dealer_trunc(P, DSEED, d.next_tag(), M * N)
    return s


# ---------------------------------------------------------------- one pass
def run(s):
    c, kind = s["c"], s["kind"]
    if kind == "matmul":
        z = c.beaver_matmul(s["x"], s["y"], s["t"], FRAC)
        return [z.s0, z.s1]
    if kind == "mul":
        z = c.beaver_mul(s["x"], s["y"], s["t"], FRAC)
        return [z.s0, z.s1]
    if kind == "mlp":
        h = c.share(s["x"], 0, s["tag"])
        for w, t, sq in s["layers"]:
            h = c.beaver_matmul(h, w, t, FRAC)
            if sq is not None:
                h = c.beaver_mul(h, None, sq, FRAC)
        return [c.reveal(h), h.s0, h.s1]
    if kind == "prepacked":
        x = c.share(s["x"], 0, s["tag"])
        z = c.beaver_matmul_prepacked(x, s["y"], s["t"], s["packed"], FRAC)
        return [c.reveal(z), z.s0, z.s1]
    if kind == "deal":
        t = c.dealer(mpc.TRIPLE_MATMUL, DSEED, s["tag"], s["dims"])
        return [t.a0, t.a1, t.b0, t.b1, t.c0, t.c1]
    if kind == "conv":
        z = c.beaver_conv1d(s["x"], s["w"], s["t"], s["stride"], FRAC)
        return [z.s0, z.s1]
    if kind == "grouped":
        if s["graph"] is not None:
            c.graph_launch(s["graph"])
        else:
            c.beaver_matmul_grouped(s["probs"], FRAC, outs=s["outs"])
        return s["flat"]
    if kind == "relu":
        z = c.relu(s["x"], s["tag"], s["t"], s["rb"], s["ra"], s["m"])
        return [z.s0, z.s1]
    z = c.mp_beaver_matmul(s["x"], s["y"], s["t"])
    return c.mp_truncate(z, FRAC, s["r"], s["theta"]).shares


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    """Bytes: shares and triples in, shares out, once each (8 bytes an element).  Operations: a ring multiply and an
    add per term of every matrix product (each party's finish is one product over 2K; the dealer's is one over K)."""
    kind = case["kind"]

    def beaver(M, N, K, P=2):
        return 8.0 * P * (2 * M * K + 2 * K * N + 2 * M * N), 2.0 * P * M * N * 2 * K

    if kind == "mul":
        n = case["n"]
        return {"bytes": (64.0 if case["square"] else 96.0) * n, "flops": (6.0 if case["square"] else 16.0) * n}
    if kind == "relu":
        return {"bytes": 86 * 8.0 * case["n"], "flops": 300.0 * case["n"]}
    if kind == "deal":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 16.0 * (M * K + K * N + M * N), "flops": 2.0 * M * N * K}
    if kind == "conv":
        cin, cout, k, stride, L = CONV[case["layer"]]
        B, lout = case["batch"], (L - k) // stride + 1
        return {"bytes": 8.0 * 2 * (2 * B * cin * L + 2 * cout * cin * k + 2 * B * cout * lout),
                "flops": 8.0 * cout * B * lout * cin * k}
    if kind == "mlp":
        B, nbytes, ops = case["batch"], 24.0 * case["batch"] * MLP[0], 0.0
        for i, (K, N) in enumerate(zip(MLP, MLP[1:])):
            b, f = beaver(B, N, K)
            nbytes, ops = nbytes + b + (64.0 if i + 2 < len(MLP) else 24.0) * B * N, ops + f
        return {"bytes": nbytes, "flops": ops}
    if kind == "grouped":
        both = [beaver(*s) for s in _group_shapes(case)]
        return {"bytes": sum(b for b, _ in both), "flops": sum(f for _, f in both)}
    M, N, K = case["M"], case["N"], case["K"]
    if kind == "party":
        b, f = beaver(M, N, K, case["P"])
        return {"bytes": b + 32.0 * case["P"] * M * N, "flops": f}
    b, f = beaver(M, N, K)
    return {"bytes": b + (24.0 * (M * K + M * N) if kind == "prepacked" else 0.0), "flops": f}


def exact(case, seed):
    """Shares of an element-wise product in plain int64 arithmetic (it wraps, as the ring does).  The other cases
    return None: their outputs are whole numbers too, and no plain 64-bit integer matrix product is at hand here."""
    if case["kind"] != "mul":
        return None
    s = prepare(case, seed)
    x, t = s["x"], s["t"]
    eps = (x.s0 - t.a0) + (x.s1 - t.a1)
    if case["square"]:
        z = [t.b0 + 2 * eps * t.a0 + eps * eps, t.b1 + 2 * eps * t.a1]
    else:
        y = s["y"]
        delta = (y.s0 - t.b0) + (y.s1 - t.b1)
        z = [t.c0 + eps * t.b0 + t.a0 * delta + eps * delta, t.c1 + eps * t.b1 + t.a1 * delta]
    return [v >> FRAC for v in z]

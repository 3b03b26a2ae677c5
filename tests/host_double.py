"""Drives the library's host code without a GPU: csrc/api.cpp linked with tests/host_double.cpp, which logs the
launches a call would make.  Operands are addresses that nothing reads."""
import ctypes
import functools
import os
import subprocess
import tempfile

import paper_2109_00984_amd as m

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PKG = os.path.join(ROOT, "paper_2109_00984_amd")
_dir = tempfile.TemporaryDirectory(prefix="host_double")  # removed when the process ends


@functools.lru_cache(None)
def library():
    out = os.path.join(_dir.name, "libhost_double.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++20", "-O1", "-w", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                    "-D__align__(n)=__attribute__((aligned(n)))", "-DHIP_SYMBOL(x)=(&(x))", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"), os.path.join(PKG, "csrc", "api.cpp"),
                    os.path.join(HERE, "host_double.cpp"), "-o", out, "-L", PKG, "-l:libmpc.so", "-Wl,-rpath," + PKG,
                    "-Wl,-Bsymbolic", "-Wl,--no-undefined"], check=True)
    lib = ctypes.CDLL(out)
    lib.double_log.restype = ctypes.c_char_p
    lib.mpc_packed_triple_bytes.restype = ctypes.c_size_t
    lib.mpc_packed_triple_bytes.argtypes = [ctypes.c_int64] * 3
    return lib


VP, I64, U64 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_uint64


class Double:
    """A context over the stand-in; every call returns its launches as (name, fields) pairs."""

    def __init__(self, limit=288 << 30):
        self.lib, self.next = library(), 1 << 40
        self.lib.double_limit(ctypes.c_size_t(limit))
        h = VP()
        self._ok(self.lib.mpc_ctx_create(0, VP(1), VP(2), U64(1), ctypes.byref(h)))
        self.h = h

    def close(self):
        self._ok(self.lib.mpc_ctx_destroy(self.h))

    def _ok(self, st):
        if st != 0:
            raise m.MPCError(st, "call")

    def array(self, *shape):
        n = 1
        for s in shape:
            n *= s
        at, self.next = self.next, self.next + (n * 8 + 511) // 256 * 256
        return at

    def arrays(self, k, *shape):
        return [VP(self.array(*shape)) for _ in range(k)]

    def triple(self, a, b, c):
        return m.Triple(*self.arrays(2, *a), *self.arrays(2, *b), *self.arrays(2, *c))

    def call(self, name, *args):
        self.lib.double_clear()
        self._ok(getattr(self.lib, name)(self.h, *args))
        out = []
        for line in self.lib.double_log().decode().splitlines():
            name, *f = line.split()
            out.append((name, {k: int(v) for k, v in (x.split("=") for x in f)}))
        return out

    def counts(self):
        v = (ctypes.c_size_t * 5)()
        self.lib.double_counts(v)
        return dict(zip(("mallocs", "refused", "frees", "syncs", "used"), v))

    def stats(self):
        s = m.Stats()
        self._ok(self.lib.mpc_ctx_stats(self.h, ctypes.byref(s)))
        return {k: int(getattr(s, k)) for k, _ in m.Stats._fields_}

    # ---------------------------------------------------------- the calls
    def matmul(self, M, N, K, form="auto", name="mpc_beaver_matmul"):
        return self.call(name, I64(M), I64(N), I64(K), *self.arrays(2, M, K), *self.arrays(2, K, N),
                         ctypes.byref(self.triple((M, K), (K, N), (M, N))), 16, m.FORMS[form], *self.arrays(2, M, N))

    def packed(self, M, N, K):
        return VP(self.array((self.lib.mpc_packed_triple_bytes(M, N, K) + 7) // 8))

    def prepacked(self, M, N, K):
        return self.call("mpc_beaver_matmul_prepacked", I64(M), I64(N), I64(K), *self.arrays(2, M, K), *self.arrays(2, K, N),
                         ctypes.byref(self.triple((M, K), (K, N), (M, N))), self.packed(M, N, K), 16, *self.arrays(2, M, N))

    def grouped(self, shapes, form="auto", packed=False):
        d = (m.MatmulDesc * len(shapes))()
        for q, (M, N, K) in zip(d, shapes):
            q.M, q.N, q.K = M, N, K
            q.x0, q.x1, q.y0, q.y1 = *self.arrays(2, M, K), *self.arrays(2, K, N)
            q.t = self.triple((M, K), (K, N), (M, N))
            q.z0, q.z1 = self.arrays(2, M, N)
        if packed:
            pk = (VP * len(shapes))(*[self.packed(*s) for s in shapes])
            return self.call("mpc_beaver_matmul_grouped_prepacked", ctypes.c_size_t(len(shapes)), d, pk, 16)
        return self.call("mpc_beaver_matmul_grouped", ctypes.c_size_t(len(shapes)), d, 16, m.FORMS[form])

    def ring(self, M, N, K, form="auto"):
        return self.call("mpc_ring_gemm", I64(M), I64(N), I64(K), *self.arrays(1, M, K), *self.arrays(1, K, N), *self.arrays(1, M, N),
                         m.FORMS[form])

    def deal(self, M, N, K):
        return self.call("mpc_dealer_triples", m.TRIPLE_MATMUL, U64(1), U64(2), (I64 * 3)(M, N, K),
                         ctypes.byref(self.triple((M, K), (K, N), (M, N))))

    def deal_packed(self, M, N, K):
        return self.call("mpc_dealer_triples_packed", U64(1), U64(2), I64(M), I64(N), I64(K),
                         ctypes.byref(self.triple((M, K), (K, N), (M, N))), self.packed(M, N, K))

    def _conv(self, B, cin, L, cout, k, s):
        lout = (L - k) // s + 1
        return (B, cin, L), (cout, cin, k), (B, cout, lout)

    def conv(self, B, cin, L, cout, k, s, form="auto"):
        x, w, z = self._conv(B, cin, L, cout, k, s)
        return self.call("mpc_beaver_conv1d", (I64 * 6)(B, cin, L, cout, k, s), *self.arrays(2, *x), *self.arrays(2, *w),
                         ctypes.byref(self.triple(x, w, z)), 16, m.FORMS[form], *self.arrays(2, *z))

    def deal_conv(self, B, cin, L, cout, k, s):
        return self.call("mpc_dealer_triples", m.TRIPLE_CONV1D, U64(1), U64(2), (I64 * 6)(B, cin, L, cout, k, s),
                         ctypes.byref(self.triple(*self._conv(B, cin, L, cout, k, s))))

    def party(self, P, M, N, K, form="auto"):
        t = m.MpTriple()
        for name, shape in (("a", (M, K)), ("b", (K, N)), ("c", (M, N))):
            for p in range(P):
                getattr(t, name)[p] = self.array(*shape)
        x, y, z = ((VP * P)(*self.arrays(P, *s)) for s in ((M, K), (K, N), (M, N)))
        return self.call("mpc_mp_beaver_matmul", P, I64(M), I64(N), I64(K), x, y, ctypes.byref(t), m.FORMS[form], z)


def form(log):
    """The form of a call's product: residue, limb, small (one launch) or plain; of several, in that order."""
    names = [n for n, _ in log]
    got = [f for f, key in (("residue", "res"), ("limb", "limb"), ("small", "small"), ("plain", "plain")) if key in names]
    return "+".join(got) or "none"


def tiles(log):
    """The residue GEMM's tile shapes."""
    return sorted({(f["bm"], f["bn"]) for n, f in log if n == "res"}, reverse=True)

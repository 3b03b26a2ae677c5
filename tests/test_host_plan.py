"""Which kernels a call launches, from the library's own host code without a GPU (tests/host_double.py)."""
import ctypes
import math
import random

import pytest

import paper_2109_00984_amd as m
import tests.test_gpu_residue as residue
import tests.test_gpu_residue_tiles as residue_tiles
from tests.host_double import Double, form, tiles


@pytest.fixture()
def d():
    c = Double()
    yield c
    c.close()


# ---------------------------------------------------------------- the one-launch kernel
@pytest.mark.parametrize("M,N,K,small", [(1, 1, 1, True), (256, 256, 1, True), (512, 512, 1, True), (512, 513, 1, False), (1024, 1024, 1, False),
                                         (1000, 1000, 3, False), (3031, 518, 2, False), (449, 591, 5, False), (32, 32768, 1, False),
                                         (16, 16384, 8, True), (16, 100000, 1, True), (100000, 16, 1, False), (100000, 8, 1, True), (16384, 16, 1, True), (262144, 1, 1, True), (1, 262144, 4, True), (512, 512, 12, True),
                                         (128, 128, 111, True), (128, 128, 112, True), (128, 192, 128, True), (128, 193, 128, False),
                                         (3072, 1, 1024, True), (16, 16, 1025, False)])
def test_one_launch_only_where_its_workgroups_pay(d, M, N, K, small):
    """Its time is that of its 4 x 4 blocks where k is short: not for many of them (1000 x 1000 x 3 took 247 us in it,
    23 in the plain form)."""
    for f in ("auto", "plain"):
        log = d.matmul(M, N, K, f)
        assert (form(log) == "small") == small, (f, log)
        assert not small or len(log) == 1


def test_one_launch_single_rows(d):
    """AUTO counts rows to a multiple of four beyond k of 48, where the kernel shares the columns' loads among them."""
    assert form(d.matmul(1, 65536, 48)) == "small" and form(d.matmul(1, 32768, 49)) == "limb"
    assert form(d.matmul(1, 32768, 49, "plain")) == "small"
    assert form(d.matmul(1, 1536, 1024)) == "small" and form(d.matmul(1, 1540, 1024)) == "limb"
    assert form(d.matmul(1, 1540, 1024, "plain")) == "small"


# ---------------------------------------------------------------- k below 16
@pytest.mark.parametrize("M,N,K,beaver,ring,deal,party", [
    (2048, 2048, 4, "plain", "plain", "limb", "plain"), (4096, 4096, 8, "plain", "plain", "limb", "plain"),
    (4096, 4096, 9, "limb", "plain", "limb", "limb"), (2048, 2048, 15, "limb", "plain", "limb", "limb"),
    (16, 100000, 15, "limb", "limb", "limb", "limb"), (64, 200000, 12, "limb", "limb", "limb", "limb"),
    (95, 50000, 8, "limb", "limb", "limb", "plain"), (96, 43691, 8, "plain", "plain", "limb", "plain"),
    (96, 43690, 8, "limb", "limb", "limb", "plain"), (512, 4096, 8, "limb", "limb", "limb", "plain"),
    (1, 4000000, 3, "limb", "limb", "limb", "plain"), (1024, 1024, 1, "plain", "plain", "plain", "plain"),
    (2048, 2048, 0, "plain", "plain", "plain", "plain"), (2048, 2048, 16, "limb", "limb", "limb", "limb")])
def test_short_k(d, M, N, K, beaver, ring, deal, party):
    """AUTO below k of 16 (16 x 100000 x 15 took 154 us in the plain form, 82 in the limb form)."""
    assert form(d.matmul(M, N, K)) == beaver
    assert form(d.ring(M, N, K)) == ring
    assert form(d.deal(M, N, K)) == deal
    assert form(d.party(3, M, N, K)) == party


@pytest.mark.parametrize("conv,online,dealt", [((8, 3, 8000, 64, 5, 1), "limb", "limb"), ((8, 1, 160000, 32, 9, 4), "limb", "limb"),
                                               ((8, 1, 16000, 64, 15, 1), "limb", "limb"), ((8, 1, 16000, 512, 3, 1), "plain", "limb"),
                                               ((64, 1, 4000, 128, 7, 1), "plain", "limb"), ((1, 1, 160, 32, 15, 1), "plain", "plain")])
def test_short_k_convolutions(d, conv, online, dealt):
    assert form(d.conv(*conv)) == online and form(d.deal_conv(*conv)) == dealt


# ---------------------------------------------------------------- tuned schedules
def shapes_key(shapes):
    """The hash that the tuned schedules' file keeps a shape list under (FNV-1a over 64-bit words)."""
    h = 1469598103934665603
    for v in [len(shapes)] + [v for s in shapes for v in s]:
        for b in v.to_bytes(8, "little"):
            h = (h ^ b) * 1099511628211 % 2**64
    return h


GROUP = [(300, 220, 500), (2040, 1040, 2512), (17, 200, 300), (1500, 2104, 3003), (40, 600, 64), (1825, 2281, 2304)]


@pytest.mark.parametrize("packed", [False, True])
def test_tuned_schedules_of_a_mixed_group(d, tmp_path, packed):
    """A group some of whose products take the residue form runs the others in the schedules tuned for the group."""
    order = sorted(GROUP, key=lambda s: -s[2])  # as the call issues them
    path = tmp_path / "tuned"
    path.write_text(f"{shapes_key(order):016x} 3 4 0 12 16 1 13 16 1\n")
    log = d.grouped(GROUP, packed=packed)
    assert form(log) == "residue+limb" and {f["variant"] for n, f in log if n == "limb"} == {14}
    d.call("mpc_autotune_load", ctypes.c_char_p(str(path).encode()))
    log = d.grouped(GROUP, packed=packed)
    assert form(log) == "residue+limb"
    got, sched = {}, None
    for n, f in log:
        if n == "limb":
            sched = (f["variant"], f["group_m"], f["remap"])
        elif n == "limb_problem":
            got[(f["M"], f["N"])] = sched
    assert got == {(17, 200): (12, 16, 1), (300, 220): (3, 4, 0), (40, 600): (3, 4, 0)}


# ---------------------------------------------------------------- memory that the device does not have
MB = 1 << 20


def test_refused_residue_workspace_is_not_asked_for_again():
    """2048^3 takes 604 MB of workspace in the residue form and 201 in the limb form."""
    d = Double(limit=500 * MB)
    assert form(d.matmul(2048, 2048, 2048)) == "limb" and d.counts()["refused"] > 0
    for _ in range(2):
        assert form(d.matmul(2048, 2048, 2048)) == "limb" and form(d.prepacked(2048, 2048, 2048)) == "limb"
        c = d.counts()
        assert c["mallocs"] == c["frees"] == c["syncs"] == 0
    d.lib.double_limit(ctypes.c_size_t(2000 * MB))  # memory is free again
    assert form(d.matmul(2048, 2048, 2048)) == "residue"
    d.close()


def test_workspace_without_the_slack():
    """The workspace grows by a quarter more than asked where that can be had."""
    d = Double(limit=700 * MB)
    assert form(d.matmul(2048, 2048, 2048)) == "residue"
    d.close()


def test_refused_growth_keeps_the_workspace():
    d = Double()
    d.matmul(1024, 1024, 1024, "limb8")
    used = d.counts()["used"]
    with pytest.raises(m.MPCError):
        d.call("mpc_reserve", ctypes.c_size_t(1 << 46))
    assert d.counts()["used"] == used
    d.call("mpc_graph_begin")
    assert form(d.matmul(1024, 1024, 1024, "limb8")) == "limb"  # no room to grow under a capture
    g = ctypes.c_void_p()
    d.call("mpc_graph_end", ctypes.byref(g))
    d._ok(d.lib.mpc_graph_destroy(g))
    # a call that has no other way asks every time
    for _ in range(2):
        with pytest.raises(m.MPCError):
            d.call("mpc_reserve", ctypes.c_size_t(1 << 46))
        assert d.counts()["refused"] > 0
    d.close()


def test_refused_slices_are_not_asked_for_again():
    d = Double()
    d.call("mpc_reserve", ctypes.c_size_t(400 * MB))
    d.lib.double_limit(ctypes.c_size_t(d.counts()["used"] + 2 * MB))
    for first in (True, False):
        log = d.matmul(500, 1100, 1000, "limb8")
        assert form(log) == "limb" and "reduce" not in [n for n, _ in log]
        assert (d.counts()["mallocs"] > 0) == first
    d.lib.double_limit(ctypes.c_size_t(2000 * MB))
    assert "reduce" in [n for n, _ in d.matmul(500, 1100, 1000, "limb8")]
    d.close()


def test_refused_limb_workspace_falls_back_to_plain():
    d = Double(limit=5 * MB)
    for first in (True, False, False):
        assert form(d.matmul(300, 300, 300)) == "plain"
        assert first or d.counts()["refused"] == d.counts()["syncs"] == 0
    with pytest.raises(m.MPCError):
        d.matmul(300, 300, 300, "limb8")
    d.close()


# ---------------------------------------------------------------- what a context counts
def profile(d):
    t = [m.GemmTiming() for _ in range(3)]
    d.call("mpc_profile_read", *[ctypes.byref(g) for g in t])
    return {n: (int(g.launches), float(g.ring_macs)) for n, g in zip(("limb8", "plain", "fp64limb"), t)}


@pytest.mark.parametrize("M,N,K,f", [(128, 128, 128, "plain"), (64, 32, 128, "auto"), (300, 200, 100, "plain"), (500, 500, 40, "plain"), (300, 200, 100, "limb8")])
def test_every_finish_is_counted_and_timed(d, M, N, K, f):
    """Two GEMM problems over the summed k, recorded under the form that ran (the one launch as the plain form)."""
    d.call("mpc_profile_enable", 1)
    before = d.stats()["gemm_problems"]
    log = d.matmul(M, N, K, f)
    assert d.stats()["gemm_problems"] - before == 2
    ran = "limb8" if form(log) == "limb" else "plain"
    assert profile(d) == {n: (1, 2.0 * M * N * 2 * K) if n == ran else (0, 0.0) for n in ("limb8", "plain", "fp64limb")}
    # a call that may not allocate makes no events
    d.matmul(64, 32, 128, name="mpc_beaver_matmul_noalloc")
    assert d.stats()["gemm_problems"] - before == 4 and profile(d)["plain"][0] == 0


# ---------------------------------------------------------------- k slices
@pytest.mark.parametrize("shapes,want", [([(250, 90, 4000 - 200 * i) for i in range(8)], {(250, 90): 6}),  # 128 tiles of up to 126 k steps: one a unit is 2
                                         ([(250, 90, 1200 - 50 * i) for i in range(8)], {(250, 90): 2}), ([(60, 64, 4000 - 200 * i) for i in range(8)], {(60, 64): 16}),
                                         ([(27, 159, 312), (64, 17, 422), (286, 23, 278), (17, 490, 3533), (165, 84, 45), (24, 181, 1511)],
                                          {(17, 490): 20, (24, 181): 12, (64, 17): 3, (27, 159): 2, (286, 23): 2, (165, 64): 1})])
def test_slices_of_uneven_groups(d, shapes, want):
    """Products of different k: the longest one's slices do not end long after the rest."""
    got = {(f["M"], f["N"]): f["slices"] for n, f in d.grouped(shapes, "limb8") if n == "limb_problem"}
    assert {k: got[k] for k in want} == want


# ---------------------------------------------------------------- the residue form's plan
def res_problems(log):
    return [f for n, f in log if n == "res_problem"]


def check_plan(log, products):
    """Every product's every chunk of k and modulus is computed once, by tiles that cover the output and stay inside its
    padded residues; the chunks cut the k range without a gap into at most 173 blocks of 64 each; the launches' tile
    lists are the problems'."""
    outs = [f for n, f in log if n == "combine_out"]
    assert len(outs) == products
    seen = {}
    for f in res_problems(log):
        assert f["end"] - f["start"] == f["nm"] * f["ntm"] * f["ntn"] and f["nm"] > 0
        seen.setdefault(f["R"], []).append(f)
    for n, f in log:
        if n == "res":
            assert f["tiles"] == sum(p["end"] - p["start"] for p in res_problems(log) if (p["bm"], p["bn"]) == (f["bm"], f["bn"]))
            assert 1 <= f["grid"] <= f["tiles"]
    pad = lambda v: -(-v // 256) * 256  # noqa: E731
    for o in outs:
        at = 0
        for ch in range(o["nch"]):
            probs = seen.pop(o["R"] + ch * o["pc"])
            assert sorted(i for f in probs for i in range(f["m0"], f["m0"] + f["nm"])) == list(range(18))
            assert len({(f["kb_begin"], f["kb_end"]) for f in probs}) == 1
            f = probs[0]
            assert f["kb_begin"] == at and 0 < f["kb_end"] - at <= 173
            at = f["kb_end"]
            for f in probs:
                assert o["M"] <= f["ntm"] * f["bm"] <= pad(o["M"]) and o["N"] <= f["ntn"] * f["bn"] <= pad(o["N"])
                assert f["pr"] == pad(o["M"]) * pad(o["N"]) and f["n64"] == pad(o["N"]) // 64
                assert f["pa"] == pad(o["M"]) * 64 * f["kbs"]
        assert at in (f["kbs"], 2 * f["kbs"])
    assert not seen


def random_shapes(seed, n, lo, hi):
    rng = random.Random(seed)
    return [tuple(int(round(math.exp(rng.uniform(math.log(a), math.log(b))))) for a, b in zip(lo, hi)) for _ in range(n)]


def test_residue_plan_covers_every_product(d):
    found = set()
    for M, N, K in random_shapes(7, 400, (200, 200, 1000), (5000, 5000, 30000)):
        for log, products in ((d.matmul(M, N, K), 2), (d.ring(M, N, K), 1), (d.deal(M, N, K), 1), (d.party(3, M, N, K), 3)):
            if form(log) == "residue":
                check_plan(log, products)
                found.update(tiles(log))
    assert found == {(256, 256), (256, 128), (128, 256), (128, 128)}


def test_residue_plan_of_groups(d):
    taken = 0
    for seed in range(12):
        shapes = random_shapes(seed, 5, (300, 300, 1000), (3000, 3000, 9000))
        log = d.grouped(shapes)
        n = len([1 for name, _ in log if name == "combine_out"])
        if n:
            check_plan(log, n)
            taken += n
    assert taken > 20


def test_residue_plan_of_convolutions(d):
    direct = 0
    for B, cin, L, cout, k, s in random_shapes(9, 300, (1, 40, 200, 128, 1, 1), (8, 600, 2000, 2500, 48, 3)):
        log = d.conv(B, cin, L, cout, k, s)
        if form(log) == "residue":
            check_plan(log, 2)
            direct += res_problems(log)[0]["ksz"] > 0
    assert direct > 30


@pytest.mark.parametrize("conv,online,dealt", [((1, 176, 93, 2311, 38, 1), "limb", "limb"), ((4, 347, 47, 1165, 35, 1), "limb", "limb"),
                                               ((4, 454, 99, 1628, 21, 3), "limb", "limb"), ((2, 555, 218, 1217, 35, 1), "limb", "limb"),
                                               ((16, 565, 69, 235, 40, 3), "limb", "limb"), ((8, 250, 777, 250, 7, 1), "residue", "residue"),
                                               ((8, 250, 735, 2000, 32, 1), "residue", "residue"), ((1, 250, 777, 250, 7, 1), "limb", "limb"),
                                               ((8, 512, 400, 512, 3, 1), "residue", "residue")])
def test_convolutions_of_few_columns(d, conv, online, dealt):
    """The residue form only where it is faster (2311 x 56 x 6688 took 668 us in it, 303 in the limb form)."""
    assert form(d.conv(*conv)) == online and form(d.deal_conv(*conv)) == dealt


# ---------------------------------------------------------------- the forms that the GPU tests of the residue form cover
def cases(test):
    """The argument lists of a parametrised test, by its parameters' names."""
    return {mark.args[0]: mark.args[1] for mark in test.pytestmark if mark.name == "parametrize"}


def test_forms_of_the_gpu_tests(d):
    for s in cases(residue.test_ring_gemm_matches_plain)["M,N,K"] + [(2500, 2305, 4161)]:
        assert form(d.ring(*s)) == "residue", s
    for *s, _ in cases(residue.test_beaver_matmul_matches_plain)["M,N,K,trunc"]:
        assert {form(d.matmul(*s)), form(d.prepacked(*s)), form(d.grouped([s]))} == {"residue"}, s
    for s in cases(residue.test_dealt_packed_operands)["M,N,K"]:
        assert form(d.deal_packed(*s)) == "residue", s
    for P in cases(residue.test_multiparty_matches_plain)["P"]:
        assert form(d.party(P, 2060, 2100, 2400)) == "residue"
    assert form(d.grouped(GROUP)) == "residue+limb"
    convs = cases(residue.test_conv_matches_plain)["B,cin,L,cout,k,s"]
    # (three of the convolutions there take the limb form)
    assert [form(d.conv(*s)) for s in convs].count("residue") == 5


@pytest.mark.parametrize("shape,want", residue_tiles.MATMULS)
def test_tiles_of_the_gpu_tests(d, shape, want):
    log = d.matmul(*shape)
    assert form(log) == "residue" and tiles(log) == want


@pytest.mark.parametrize("shape,want,chunks,mid", residue_tiles.CONVS)
def test_convolutions_of_the_gpu_tests(d, shape, want, chunks, mid):
    log = d.conv(*shape)
    probs = res_problems(log)
    assert form(log) == "residue" and tiles(log) == want
    if chunks is None:
        assert all(f["ksz"] == 0 for f in probs)
        return
    assert all(f["ksz"] == shape[4] and f["stride"] == shape[5] for f in probs)
    assert len({f["kb_begin"] for f in probs}) == chunks
    assert any(f["kb_begin"] % f["kbs"] % f["ksz"] for f in probs) == mid


@pytest.mark.parametrize("shape,want,direct", residue_tiles.DEALT)
def test_dealt_convolutions_of_the_gpu_tests(d, shape, want, direct):
    log = d.deal_conv(*shape)
    assert form(log) == "residue" and tiles(log) == want and all((f["ksz"] > 0) == direct for f in res_problems(log))


# ---------------------------------------------------------------- many parties
@pytest.mark.parametrize("P,M,N,K,eager,captured", [(8, 74, 10, 30, "fused", "fused"), (9, 74, 10, 30, "fused", "jobs"), (16, 237, 3, 191, "jobs", "jobs"),
                                                    (16, 32, 70, 100, "fused", "jobs"), (16, 100, 400, 600, "fused", "fused"), (12, 200, 200, 200, "jobs", "jobs")])
def test_many_party_packs(P, M, N, K, eager, captured):
    """Few blocks of many parties: a pack job per party where the launches are not waited for (16 parties' 237 x 3 x 191
    40 us, in the fused pack's chain 52)."""
    d = Double()
    packs = lambda log: "fused" if "limb_pack_party" in [n for n, _ in log] else "jobs"  # noqa: E731
    d.call("mpc_reserve", ctypes.c_size_t(1 << 20))
    log = d.party(P, M, N, K, "limb8")
    assert form(log) == "limb" and packs(log) == eager
    if eager == "jobs":
        assert [f["set"] for n, f in log if n == "limb_pack"] == [9, 9] and [n for n, _ in log].count("mp_open") == 2
        assert sum(f["jobs"] for n, f in log if n == "limb_pack") == 2 * P + 2
    d.call("mpc_graph_begin")  # the eager call made the workspace that this needs
    assert packs(d.party(P, M, N, K, "limb8")) == captured
    g = ctypes.c_void_p()
    d.call("mpc_graph_end", ctypes.byref(g))
    d._ok(d.lib.mpc_graph_destroy(g))
    d.close()

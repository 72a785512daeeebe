"""How a backward is cut into workgroups (csrc/plan.hpp, plain C++): the plan that is found by bisection is the one that a search step by
step finds."""
import ctypes
import math
import os
import random
import shutil
import subprocess

import pytest

import paper_2603_00040_amd as aq
from paper_2603_00040_amd import build as B

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not on PATH")


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = str(d / "plan.cpp"), str(d / "plan.so")
    with open(src, "w") as f:
        f.write('#include "plan.hpp"\n'
                'extern "C" void plan(int q, int kv, int L, int d, int causal, int cus, long long* o) {\n'
                '    const aq::BwdPlan p = aq::plan_backward(q, kv, L, d, causal != 0, cus);\n'
                '    o[0] = p.joint; o[1] = p.splits; o[2] = p.iters; o[3] = (long long)p.part_bytes; o[4] = p.dq_first;\n'
                '}\n'
                'extern "C" int in_pairs(int q, int kv, int L, int d, int causal, int cus) {\n'
                '    return aq::joint_in_pairs(aq::plan_backward(q, kv, L, d, causal != 0, cus), q, kv, L, d, causal != 0, cus);\n'
                '}\n'
                'extern "C" int few(int q, int kv, int L, int causal, int pieces, int cus) { return aq::few_rows(q, kv, L, causal != 0, pieces != 0, cus); }\n')
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", B.CSRC, src, "-o", lib], check=True)
    L = ctypes.CDLL(lib)
    out = (ctypes.c_longlong * 5)()

    def plan(*a):
        L.plan(*a, out)
        return tuple(out)
    plan.in_pairs = lambda *a: bool(L.in_pairs(*a))
    plan.few = lambda *a: bool(L.few(*a))
    return plan


def _step_by_step(BHq, BHkv, L, d, causal, cus):
    Lp = -(-L // 128) * 128
    nt, G, nq32 = Lp // 128, BHq // BHkv, -(-L // 32)
    n8q, n8kv = BHq * -(-Lp // 256), BHkv * -(-Lp // 256)
    fill = lambda n: n / (-(-n // cus) * cus)  # noqa: E731
    if (Lp >= 32768 and n8kv >= 2 * cus) if causal else (n8kv >= 2 * cus and fill(n8q) + fill(n8kv) >= 2 * 0.97):
        return 0, 1, 0, 0, 0
    whole = nq32 * G
    dq_longest = 1.16 * (Lp // 64)
    dq_mean = 0.5 * dq_longest if causal else dq_longest
    W = nt * (BHkv * (G * (nq32 - 2.0 * (nt - 1) if causal else float(nq32))) + BHq * dq_mean) / cus
    T, ndq = max(0.45 * W, 0.6 * dq_mean, 4.0), BHq * nt
    room = 2 * cus - (ndq if ndq < cus else 0)
    tiles = [(nq32 - (4 * kt if causal else 0)) * G for kt in range(nt)]
    while T < whole and sum(-(-n // int(T)) for n in tiles) * BHkv > room:
        T = T * 1.04 + 1.0
    if T >= whole:
        return 1, 1, whole, 0, int(dq_longest > 1.5 * whole)
    splits = -(-whole // int(T))
    return 1, splits, int(T), BHkv * nt * splits * 2 * 128 * d * 4, int(dq_longest > 1.5 * int(T))


def test_bisection_finds_the_plan_of_a_search_step_by_step(planner):
    rng = random.Random(0)
    shapes = [(1, 1, 30000, 128, 1, 256), (1, 1, 1, 64, 0, 256), (32, 8, 777, 128, 1, 256), (40, 40, 75600, 128, 0, 256), (32, 4, 3001, 128, 1, 256)]
    for _ in range(1500):
        kv = rng.choice([1, 1, 2, 3, 8, 12, 40])
        L = int(math.exp(rng.uniform(0.0, math.log(66000))))
        shapes.append((kv * rng.choice([1, 1, 2, 4, 8, 71]), kv, L, rng.choice([64, 128]), rng.randint(0, 1), rng.choice([256, 256, 32, 64])))
    split = 0
    for s in shapes:
        p = planner(*s)
        assert p == _step_by_step(*s), s
        split += p[1] > 1
        if p[1] > 1:        # the pieces of a key tile fit the room that the plan states
            assert p[2] >= 4 and p[3] == s[1] * (-(-s[2] // 128)) * p[1] * 2 * 128 * s[3] * 4
    assert split > 400


def test_largest_shapes_are_planned_without_overflow(planner):
    for s in ((65535, 1, 1, 128, 1, 256), (65535, 1, 1 << 14, 64, 1, 256), (1, 1, 1 << 20, 128, 1, 256), (1, 1, 1 << 20, 128, 0, 256), (512, 1, 65536, 128, 1, 256)):
        joint, splits, iters, part, _ = planner(*s)
        assert splits >= 1 and 0 <= iters <= 0x7FFFFFFF and 0 <= part <= 256 << 20, s


def test_size_query_includes_the_plan():
    """Both masks' plans fit what is asked for."""
    for B_, Hq, Hkv, L, d in ((1, 12, 12, 1560, 128), (2, 16, 4, 3001, 128), (1, 1, 1, 30000, 128)):
        size = aq.workspace_bytes(aq.WS_BWD, B_, Hq, Hkv, L, d)
        part = max(_step_by_step(B_ * Hq, B_ * Hkv, L, d, c, 256)[3] for c in (0, 1))
        Lp = -(-L // 128) * 128
        assert size >= part + 2 * (Hq + Hkv) * B_ * Lp * d * 2


def test_whole_key_tiles_of_d64_keep_to_two_workgroups(planner):
    """Long chains that end last (whole key tiles, a few more than compute units) have no third workgroup beside them; pieces, single heads
    without a mask, short rows under one, fewer tiles and whole rounds of them do."""
    for s in ((64, 8, 5518, 64, 0), (64, 8, 5000, 64, 0), (16, 4, 9637, 64, 0), (32, 8, 8456, 64, 1), (12, 12, 5781, 64, 1), (48, 12, 5673, 64, 1)):
        assert planner(*s, 256)[1] == 1 and planner.in_pairs(*s, 256), s
    for s in ((64, 16, 4096, 64, 0), (32, 16, 3300, 64, 0), (4, 4, 10205, 64, 0), (48, 48, 8700, 64, 0), (64, 8, 5518, 64, 1), (96, 96, 668, 64, 1), (48, 12, 16255, 64, 1),
              (2, 2, 256, 64, 0), (64, 8, 5518, 128, 0), (16, 2, 12000, 64, 0)):
        assert not planner.in_pairs(*s, 256), s


def test_routes_of_the_shapes_that_the_gpu_tests_name(planner):
    """Which kernel an NVFP4 backward with all the room it asks for takes: the shapes of tests/test_gpu_bwd_routes.py lie on the side of
    few_rows that they are for."""
    from tests.test_gpu_bwd_routes import CUT, FEW, SPARE

    def route(B_, Hq, Hkv, L, d, causal):
        _, splits, _, _, dq_first = planner(B_ * Hq, B_ * Hkv, L, d, causal, 256)
        Lp, align = -(-L // 128) * 128, lambda n: -(-n // 256) * 256
        nq, nk = B_ * Hq, B_ * Hkv
        small = 2 * (nq + nk) * Lp * d * 2 + align(nq * Lp * 8) + align(3 * nq * 256) + align(nk * 32 * d * 8) + align(nk * d * 4) < 2 << 20
        return planner.few(nq, nk, L, causal, splits > 1 and not small, 256), splits > 1, bool(dq_first), small
    for s in FEW:
        assert route(*s)[0], s
    for s in CUT:
        few, cut, _, small = route(*s)
        assert not few and cut and not small and s[1] == s[2], s
    assert {route(*s)[2] for s in CUT} == {False, True}
    for s in SPARE:      # cut if there were room, and small enough to be asked for without; a plain NVFP4 backward has few rows there
        few, cut, _, small = route(*s)
        assert few and cut and small, s

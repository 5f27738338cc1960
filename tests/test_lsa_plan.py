"""The tile that the one-kernel Layer Self-Attention takes (csrc/moa_lsa_plan.h: host arithmetic, compiled here with g++)."""
import ctypes as C
import random
import subprocess
from collections import namedtuple
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2410_03804_amd" / "csrc"
LDS = 160 * 1024
Plan = namedtuple("Plan", "tokens dense wide_tiles")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("lsa_plan")
    (d / "plan.cpp").write_text('#include "moa_lsa_plan.h"\nextern "C" void plan(int packed, int64_t T, int L, int d_in, int units, size_t lds, int64_t *out)\n'
                                "{\n    const moa::LsaFusedPlan p = moa::lsa_fused_plan(packed, T, L, d_in, units, lds);\n"
                                "    out[0] = p.tokens, out[1] = p.dense, out[2] = p.wide_tiles;\n}\n")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-shared", "-fPIC", f"-I{CSRC}", "-o", str(d / "plan.so"), str(d / "plan.cpp")],
                   check=True)
    f = C.CDLL(str(d / "plan.so")).plan
    f.argtypes = [C.c_int, C.c_int64, C.c_int, C.c_int, C.c_int, C.c_size_t, C.POINTER(C.c_int64)]

    def call(packed, T, L, d_in, units, lds=LDS):
        out = (C.c_int64 * 3)()
        f(packed, T, L, d_in, units, lds, out)
        return Plan(out[0], bool(out[1]), out[2])
    return call


def calls(n, seed):
    rng = random.Random(seed)
    for _ in range(n):
        yield rng.random() < 0.7, rng.randint(1, 1100), rng.randint(1, 96), 64 * rng.randint(2, 64), rng.randint(1, 40)


def test_forms_that_fill_the_lds_only_where_a_workgroup_may_have_all_of_it(plan):
    """128 and 160 rows take the last byte of 160 KB.  With less (0: the query failed) every call gets a smaller tile."""
    big = 0
    for packed, T, L, d_in, units in calls(3000, 1):
        blocks = (L + 31) // 32
        for lds in (0, 64 * 1024, LDS - 1):
            p = plan(packed, T, L, d_in, units, lds)
            assert not p.dense and p.wide_tiles == 0 and p.tokens * blocks <= 3, (packed, T, L, d_in, units, lds, p)
        p = plan(packed, T, L, d_in, units)
        big += p.dense or p.wide_tiles > 0 or p.tokens * blocks == 4
    assert big > 1000


def test_tiles_cover_the_tokens(plan):
    for packed, T, L, d_in, units in calls(3000, 2):
        p = plan(packed, T, L, d_in, units)
        assert p.tokens in {1: (2, 3, 4), 2: (1, 2), 3: (2,) if p.dense else (1,)}[(L + 31) // 32]
        assert not (p.dense or p.wide_tiles) or packed
        assert 5 * (p.wide_tiles - 1) < T, "no tile behind the last token"
        assert not p.dense or 2 * L <= 160


def test_rounds_are_those_of_the_xcd_with_the_most_units(plan):
    """Units are dealt to eight XCDs of 32 compute units: 1 .. 8 units put one on some XCD, 9 .. 16 two, so a launch takes as
    many rounds as one with the units filled up to eights, and the tile is the same."""
    for packed, T, L, d_in, units in calls(6000, 3):
        assert plan(packed, T, L, d_in, units) == plan(packed, T, L, d_in, (units + 7) // 8 * 8), (packed, T, L, d_in, units)


@pytest.mark.parametrize("T,L,units,want", [
    (32, 80, 8, Plan(1, False, 0)),         # one round of one token per workgroup
    (33, 80, 8, Plan(2, True, 0)),          # two would be needed
    (78, 80, 6, Plan(2, True, 0)),          # three rounds against two
    (32, 80, 3, Plan(1, False, 0)),
    (60, 32, 8, Plan(2, False, 0)),
    (96, 32, 3, Plan(3, False, 0)),
    (160, 32, 8, Plan(4, False, 32)),       # a round of five tokens per workgroup
    (1024, 32, 8, Plan(4, False, 0)),       # eight whole rounds of four
    (40, 64, 2, Plan(2, False, 0)),         # two rounds of 64 rows against one of 128
])
def test_packed_tiles_at_width_2048(plan, T, L, units, want):
    assert plan(True, T, L, 2048, units) == want

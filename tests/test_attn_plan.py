"""Which kernels the attention cores of a launch take (csrc/moa_attn_plan.h: host arithmetic, compiled here with g++)."""
import ctypes as C
import math
import random
import subprocess
from collections import namedtuple
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2410_03804_amd" / "csrc"
AUTO, WHOLE, SPLIT, SPLIT_WIDE = range(4)
Shape = namedtuple("Shape", "B Mq H Hkv dh")
Choice = namedtuple("Choice", "kind nsplit rows_pad wide bytes")      # kind: 0 whole key range, 1 split, 2 neither


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("attn_plan")
    (d / "plan.cpp").write_text(
        '#include "moa_attn_plan.h"\nextern "C" size_t room(int form, const int *s, int cap) { return moa::split_room(form, s[0], s[1], s[2], s[3], s[4], cap); }\n'
        'extern "C" void choose(int form, const int *s, int n, const int *cap, const int *mt, const int *mfma, const size_t *room, int pair, int64_t *out)\n{\n'
        "    moa::AttnCore c[8] = {};\n    moa::AttnChoice r[8] = {};\n    for (int i = 0; i < n; ++i) c[i] = {cap[i], mt[i], mfma[i] != 0, room[i]};\n"
        "    moa::choose_attn(form, s[0], s[1], s[2], s[3], s[4], c, n, pair != 0, r);\n"
        "    for (int i = 0; i < n; ++i) {\n        const bool split = r[i].kind == moa::AttnChoice::SPLIT;\n        int64_t *o = out + 5 * i;\n"
        "        o[0] = r[i].kind, o[1] = split ? r[i].geo.nsplit : 0, o[2] = split ? r[i].geo.rows_pad : 0, o[3] = split && r[i].geo.wide;\n"
        "        o[4] = split ? (int64_t)moa::split_bytes(r[i].geo, s[0], s[3], s[4]) : 0;\n    }\n}\n")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-O1", "-shared", "-fPIC", f"-I{CSRC}", "-o", str(d / "plan.so"), str(d / "plan.cpp")],
                   check=True)
    so = C.CDLL(str(d / "plan.so"))
    so.room.restype = C.c_size_t
    return so


def room(lib, shape, cap, form=AUTO):
    return lib.room(form, (C.c_int * 5)(*shape), cap)


def choose(lib, shape, cores, form=AUTO, pair=True):
    """cores: (P_cap, tree keys, operands fit, scratch) each"""
    n, out = len(cores), (C.c_int64 * (5 * len(cores)))()
    cap, mt, mfma = ((C.c_int * n)(*[int(c[i]) for c in cores]) for i in range(3))
    lib.choose(form, (C.c_int * 5)(*shape), n, cap, mt, mfma, (C.c_size_t * n)(*[c[3] for c in cores]), int(pair), out)
    return [Choice(out[5 * i], out[5 * i + 1], out[5 * i + 2], bool(out[5 * i + 3]), out[5 * i + 4]) for i in range(n)]


def shapes(n, seed):
    rng = random.Random(seed)
    for _ in range(n):
        Hkv = rng.choice([1, 2, 3, 4, 8])
        G = rng.choice([1, 2, 4, 7, 8, 11])
        yield rng, Shape(rng.choice([1, 2, 3, 4, 7, 8, 16]), rng.randint(1, 256), G * Hkv, Hkv, rng.choice([64, 128, 128, 128]))


def step_cores(rng, lib, shape, form, n):
    """A step's cores: the cross-attention's and verification layers' with their tree, scratch as a step hands it out (for the larger
    of the two capacities), now and then too little of it or operands of another alignment."""
    ca, ver = (int(math.exp(rng.uniform(math.log(32), math.log(40000)))) for _ in range(2))
    if rng.random() < 0.3:
        ca, ver = 8192 - rng.randint(0, 40), 8192 - shape.Mq + rng.randint(-2, 40)
    ver = max(ver, 1)
    each = room(lib, shape, max(ca, ver), form)
    give = lambda: each if rng.random() < 0.9 else rng.choice([0, 256, each // 2])
    return [(ca, 0, rng.random() < 0.97, give())] + [(ver, shape.Mq, rng.random() < 0.97, give()) for _ in range(n - 1)]


@pytest.mark.parametrize("form", [AUTO, SPLIT, SPLIT_WIDE])
def test_a_core_is_given_slices_that_its_own_scratch_holds(lib, form):
    split = 0
    for rng, shape in shapes(4000, form):
        cores = step_cores(rng, lib, shape, form, rng.randint(1, 5))
        for core, c in zip(cores, choose(lib, shape, cores, form, rng.random() < 0.7)):
            assert c.kind != 1 or (core[2] and c.bytes <= core[3]), (shape, cores, c)
            split += c.kind == 1
    assert split > 2000


def test_a_smaller_capacity_that_needs_more_scratch(lib):
    """The cross-attention over its whole key range, the verification layer in slices at 127 keys less, for which the 128-row tiles
    take 135 KB more than scratch for the cross-attention's capacity is: not in slices, rather than past the end of its scratch."""
    shape = Shape(4, 128, 11, 1, 128)
    each = room(lib, shape, 8192)
    assert room(lib, shape, 8065) > each
    got = choose(lib, shape, [(8192, 0, True, each), (8065, 128, True, each)])
    assert got[0].kind == 0 and got[1].kind == 2
    got = choose(lib, shape, [(8192, 0, True, each), (8065, 128, True, room(lib, shape, 8065))])
    assert got[0].kind == 0 and got[1].kind == 1


@pytest.mark.parametrize("form", [AUTO, SPLIT, SPLIT_WIDE])
def test_a_core_takes_the_same_whoever_is_beside_it(lib, form):
    """Alone, or as one of the first two of a step: the layers behind them change nothing, nor does their number."""
    wide = 0
    for rng, shape in shapes(2000, 10 + form):
        cores = step_cores(rng, lib, shape, form, 5)
        alone = [choose(lib, shape, [c], form)[0] for c in cores]
        pair = choose(lib, shape, cores[:2], form)
        for n in (3, 4, 5):
            assert choose(lib, shape, cores[:n], form) == pair + alone[2:n], (shape, cores)
            assert choose(lib, shape, cores[:n], form, pair=False) == alone[:n], (shape, cores)
        wide += alone[4].wide
    assert wide > 200

"""Which verification layers of a step share launches (csrc/moa_step_mem.h: host arithmetic, compiled here with g++)."""
import ctypes as C
import random
import subprocess
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2410_03804_amd" / "csrc"
LAYER = ("x", "wq", "wk", "wv", "wo", "kcache", "vcache", "out", "ktree", "vtree")
REST_READS = ("parent", "tok", "tgt", "tok_off", "prefix_len", "lsa_hs", "lsa_wq", "lsa_wk", "lsa_wv", "lsa_wo", "lsa_w_packed", "ca_wk", "ca_wv",
              "ca_wk_lsa_wo", "ca_wv_lsa_wo", "ca_xq", "ca_wq", "ca_wo")
SA = ("emb", "wq", "wk", "wv", "wo", "kcache", "vcache", "out", "k_draft", "v_draft")
INT_READS, INT_WRITES = ("parent", "tok", "tgt", "tok_off"), ("depth", "path", "n_path", "bonus", "ca_len", "dev_status")
REST_WRITES = ("mask", "depth", "path", "n_path", "bonus", "lsa_out", "ca_len", "ca_k", "ca_v", "ca_out", "dev_status")
SP, SHQ, SHKV = 70, 6, 1                                                 # the Self-Attention layer's cache capacity and heads
S = dict(L=4, d=256, H=4, Hkv=2, dh=64, din=128, Hl=2, Hkvl=2)          # bf16
B, M, P, CP, T = 2, 19, 50, 60, 7


def sizes():
    es, e, ekv, eq, el = 2, S["H"] * S["dh"], S["Hkv"] * S["dh"], S["Hl"] * S["dh"], S["Hkvl"] * S["dh"]
    d, din, R = S["d"], S["din"], B * M
    n = dict(x=R * d * es, wq=e * d * es, wk=ekv * d * es, wv=ekv * d * es, wo=e * d * es, kcache=B * P * ekv * es, vcache=B * P * ekv * es,
             out=R * d * es, ktree=R * ekv * es, vtree=R * ekv * es, parent=4 * R, tok=4 * R, tgt=4 * R, tok_off=4 * (B + 1), prefix_len=4 * B,
             lsa_hs=T * S["L"] * din * es, lsa_wq=eq * din * es, lsa_wk=el * din * es, lsa_wv=el * din * es, lsa_wo=eq * eq * es,
             lsa_w_packed=2 * eq * din * es, ca_wk=ekv * eq * es, ca_wv=ekv * eq * es, ca_wk_lsa_wo=ekv * eq * es, ca_wv_lsa_wo=ekv * eq * es,
             ca_xq=R * d * es, ca_wq=e * d * es, ca_wo=e * d * es, mask=8 * R, depth=4 * R, path=4 * R, n_path=4 * B, bonus=4 * B,
             lsa_out=T * eq * es, ca_len=4 * B, ca_k=B * CP * ekv * es, ca_v=B * CP * ekv * es, ca_out=R * d * es, dev_status=4)
    return n


def sa_sizes():
    es, e, ekv, d, R = 2, SHQ * S["dh"], SHKV * S["dh"], S["d"], B * M
    return dict(emb=R * d * es, wq=e * d * es, wk=ekv * d * es, wv=ekv * d * es, wo=e * d * es, kcache=B * SP * ekv * es, vcache=B * SP * ekv * es,
                out=R * d * es, k_draft=R * ekv * es, v_draft=R * ekv * es)


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("step_mem")
    rest = REST_READS + REST_WRITES
    arrays = {"x": "v_x_host", "wq": "v_wq_host", "wk": "v_wk_host", "wv": "v_wv_host", "wo": "v_wo_host", "kcache": "v_kcache_host",
              "vcache": "v_vcache_host", "out": "v_out_host", "ktree": "v_ktree_host", "vtree": "v_vtree_host"}
    src = '#include "moa_step_mem.h"\n' \
          'extern "C" int run(char **rest, char ***layers, int n, int l0, int most, int with_rest)\n{\n' \
          f'    moa_shape_t s = {{{S["L"]}, {S["d"]}, {S["H"]}, {S["Hkv"]}, {S["dh"]}, {S["din"]}, {S["Hl"]}, {S["Hkvl"]}, MOA_BF16}};\n' \
          f'    moa_step_args_t a = {{}};\n    a.shape = &s; a.B = {B}; a.M = a.Mq = {M}; a.P_cap = {P}; a.ca_P_cap = {CP}; a.T_lsa = {T}; a.n_verify_layers = n;\n'
    src += "".join(f"    a.{name} = (decltype(a.{name}))rest[{i}];\n" for i, name in enumerate(rest))
    src += "".join(f"    a.{arrays[name]} = (decltype(a.{arrays[name]}))layers[{i}];\n" for i, name in enumerate(LAYER))
    src += "    return moa::verify_run(&a, l0, most, with_rest);\n}\n" \
           "extern \"C\" int sa(char **rest, char ***layers, int n, char **own)\n{\n" \
           f'    moa_shape_t s = {{{S["L"]}, {S["d"]}, {S["H"]}, {S["Hkv"]}, {S["dh"]}, {S["din"]}, {S["Hl"]}, {S["Hkvl"]}, MOA_BF16}}, o = s;\n' \
           f"    o.n_q_heads = {SHQ}; o.n_kv_heads = {SHKV};\n" \
           f"    moa_step_args_t a = {{}};\n    a.shape = &s; a.sa_shape = &o; a.B = {B}; a.M = a.Mq = {M}; a.P_cap = {P}; a.sa_P_cap = {SP}; a.n_verify_layers = n;\n" \
           + "".join(f"    a.{name} = (decltype(a.{name}))rest[{i}];\n" for i, name in enumerate(rest)) \
           + "".join(f"    a.{arrays[name]} = (decltype(a.{arrays[name]}))layers[{i}];\n" for i, name in enumerate(LAYER)) \
           + "".join(f"    a.sa_{name} = (decltype(a.sa_{name}))own[{i}];\n" for i, name in enumerate(SA)) \
           + "    return moa::sa_apart(&a, n);\n}\n" \
           'extern "C" int carve(int most, size_t qa, size_t core, char *spare, size_t ns, char *idle, size_t ni, size_t *out)\n{\n' \
           "    moa::VerifyMem m[4] = {};\n    const int n = moa::carve_verify(m, most, qa, core, spare, ns, idle, ni);\n" \
           "    for (int i = 1; i < n; ++i, out += 4) out[0] = (size_t)m[i].q, out[1] = (size_t)m[i].h, out[2] = (size_t)m[i].core, out[3] = m[i].core_bytes;\n" \
           "    return n;\n}\n"
    (d / "run.cpp").write_text(src)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-Wno-unused-function", "-O1", "-shared", "-fPIC", f"-I{CSRC}", f"-I{d}", "-o",
                    str(d / "run.so"), str(d / "run.cpp")], check=True)
    so = C.CDLL(str(d / "run.so"))
    f = so.run

    def call(rest_at, layers_at, l0, most, with_rest):
        n = len(layers_at)
        r = (C.c_void_p * len(rest))(*[rest_at[k] for k in rest])
        cols = [(C.c_void_p * n)(*[la[k] for la in layers_at]) for k in LAYER]
        table = (C.c_void_p * len(LAYER))(*[C.addressof(c) for c in cols])
        return f(r, table, n, l0, most, int(with_rest))

    def carve(most, qa, core, spare, spare_bytes, idle, idle_bytes):
        """(queries, heads, core scratch, its bytes) of every layer after the first"""
        out = (C.c_size_t * 12)()
        z = C.c_size_t
        n = so.carve(most, z(qa), z(core), C.c_void_p(spare), z(spare_bytes), C.c_void_p(idle), z(idle_bytes), out)
        return [tuple(out[4 * i:4 * i + 4]) for i in range(n - 1)]
    def sa(rest_at, layers_at, own_at):
        n = len(layers_at)
        cols = [(C.c_void_p * n)(*[la[k] for la in layers_at]) for k in LAYER]
        return bool(so.sa((C.c_void_p * len(rest))(*[rest_at[k] for k in rest]), (C.c_void_p * len(LAYER))(*[C.addressof(c) for c in cols]), n,
                          (C.c_void_p * len(SA))(*[own_at[k] for k in SA])))
    call.carve, call.sa = carve, sa
    return call


def expected(rest_at, layers_at, l0, most, with_rest):
    """From the definition: byte ranges of what is read and written, pairwise."""
    n = sizes()
    span = lambda at, keys: [(at[k], at[k] + n[k]) for k in keys if at[k]]
    meet = lambda a, b: any(p < y and x < q for p, q in a for x, y in b)
    reads = [span(la, LAYER[:7]) for la in layers_at]
    writes = [span(la, LAYER[7:]) for la in layers_at]
    rr, rw = span(rest_at, REST_READS), span(rest_at, REST_WRITES)
    usable = lambda l: all(layers_at[l][k] for k in ("wq", "wk", "wv", "wo")) and all(layers_at[l][k] % 16 == 0 for k in LAYER)
    most = min(most, len(layers_at) - l0)
    if most <= 1 or not usable(l0) or (with_rest and any(rest_at[k] % 16 for k in ("ca_xq", "ca_wq", "ca_wo", "ca_k", "ca_v", "ca_out"))):
        return 1
    k = 1
    while k < most:
        l = l0 + k
        if not usable(l) or (with_rest and (meet(writes[l], rr) or meet(writes[l], rw) or meet(reads[l], rw))):
            break
        if any(meet(writes[l], reads[i]) or meet(writes[i], reads[l]) or meet(writes[l], writes[i]) for i in range(l0, l)):
            break
        k += 1
    return k


def layout(rng, n_layers):
    """Buffers one behind another, nothing shared."""
    n, at = sizes(), 1 << 24
    def place(k):
        nonlocal at
        p, at = at, at + (n[k] + 15) // 16 * 16
        return p
    rest = {k: place(k) for k in REST_READS + REST_WRITES}
    return rest, [{k: place(k) for k in LAYER} for _ in range(n_layers)]


def test_separate_buffers_share_up_to_what_there_is_room_for(run):
    rest, layers = layout(random.Random(0), 6)
    assert [run(rest, layers, 0, most, True) for most in (1, 2, 3, 4)] == [1, 2, 3, 4]
    assert run(rest, layers, 4, 4, False) == 2 and run(rest, layers, 5, 4, False) == 1


@pytest.mark.parametrize("seed", range(4))
def test_any_overlap_ends_a_run(run, seed):
    """One to three buffers moved onto (or to the edge of, or off the alignment beside) another: the rule and the definition agree."""
    rng, n = random.Random(seed), sizes()
    seen = set()
    for _ in range(400):
        layers_n = rng.randint(2, 6)
        rest, layers = layout(rng, layers_n)
        for _ in range(rng.randint(0, 3)):
            dst, key = (rng.choice(layers), rng.choice(LAYER)) if rng.random() < 0.8 else (rest, rng.choice(REST_READS + REST_WRITES))
            src, other = (rng.choice(layers), rng.choice(LAYER)) if rng.random() < 0.6 else (rest, rng.choice(REST_READS + REST_WRITES))
            kind = rng.randrange(6)
            if kind == 0: dst[key] = src[other]                                       # the same buffer
            elif kind == 1: dst[key] = src[other] + n[other] - 16 if n[other] >= 16 else src[other]      # its last piece
            elif kind == 2: dst[key] = src[other] - n[key] + 16                       # its first piece
            elif kind == 3: dst[key] = src[other] - (n[key] + 15) // 16 * 16          # up to its edge
            elif kind == 4: dst[key] += 8                                             # aligned to 8 only
            elif key in ("wq", "wk", "wv", "wo") and dst is not rest: dst[key] = 0    # already projected
        l0, most, with_rest = rng.randint(0, layers_n - 1), rng.randint(1, 4), rng.random() < 0.5
        if with_rest:
            l0 = 0
        got, want = run(rest, layers, l0, most, with_rest), expected(rest, layers, l0, most, with_rest)
        assert got == want, (rest, layers, l0, most, with_rest)
        seen.add(want)
    assert seen == {1, 2, 3, 4}


@pytest.mark.parametrize("core", [0, 512, 4096])
def test_buffers_lie_apart_in_what_they_are_carved_from(run, core):
    """Queries, heads and as much core scratch as is said to be there: each in the spare or the idle memory, none over another.
    As many layers as there is room for: a core's scratch goes to the idle memory while that lasts, then to the spare one."""
    rng, seen = random.Random(core), set()
    for _ in range(300):
        most, qa = rng.randint(1, 4), 256 * rng.randint(1, 6)
        spare, idle = (1 << 20, 256 * rng.randint(0, 120)), (1 << 24, 256 * rng.randint(0, 50))
        got = run.carve(most, qa, core, *spare, *idle)
        spans = []
        for q, h, at, there in got:
            assert there == core and (at != 0) == (core > 0)
            spans += [(q, q + qa), (h, h + qa)] + [(at, at + there)] * (there > 0)
        for lo, hi in spans:
            assert any(base <= lo and hi <= base + n for base, n in (spare, idle))
        spans.sort()
        assert all(a[1] <= b[0] for a, b in zip(spans, spans[1:]))
        in_idle = min(most - 1, idle[1] // core if core else most - 1)
        fit = min(in_idle, spare[1] // (2 * qa))
        fit += min(most - 1 - fit, max(0, spare[1] - 2 * qa * fit) // (2 * qa + core)) if fit == in_idle else 0
        assert len(got) == fit
        seen.add((len(got), any(at >= idle[0] for _, _, at, _ in got), any(0 < at < idle[0] for _, _, at, _ in got)))
    assert {n for n, _, _ in seen} == {0, 1, 2, 3}
    if core:
        assert {(3, True, False), (3, True, True), (3, False, True)} <= seen


@pytest.mark.parametrize("seed", range(3))
def test_self_attention_joins_only_apart_from_the_integer_work_and_the_layers(run, seed):
    """One or two of its buffers moved onto or to the edge of a buffer of the step, a layer or its own: the rule and the definition, byte
    ranges of what is read and written pairwise, agree.  (What lies behind the first launch of a step may meet anything of the layer's.)"""
    rng, n, own_n = random.Random(seed), sizes(), sa_sizes()
    meet = lambda a, b: any(p < y and x < q for p, q in a for x, y in b)
    joined = 0
    for _ in range(400):
        rest, layers = layout(rng, rng.randint(1, 3))
        at, own = 1 << 28, {}
        for k in SA:
            own[k], at = at, at + (own_n[k] + 15) // 16 * 16
        for _ in range(rng.randint(0, 2)):
            key, (src, other) = rng.choice(SA), rng.choice([(rest, rng.choice(REST_READS + REST_WRITES)), (rng.choice(layers), rng.choice(LAYER))])
            end = src[other] + (n[other] + 15) // 16 * 16
            own[key] = rng.choice([src[other], end, src[other] - (own_n[key] + 15) // 16 * 16, max(end - 16, src[other]), own[key] + 8])
        span = lambda where, size, keys: [(where[k], where[k] + size[k]) for k in keys]
        reads, writes = span(own, own_n, SA[:7]), span(own, own_n, SA[7:])
        mask = span(rest, n, ("mask",))
        want = not any(own[k] % 16 for k in SA) and not meet(writes, span(rest, n, INT_READS + INT_WRITES) + mask) and \
            not meet(reads, span(rest, n, INT_WRITES) + mask)
        for la in layers:
            lr, lw = span(la, n, LAYER[:7]), span(la, n, LAYER[7:])
            want = want and not meet(lw, reads + writes) and not meet(lr, writes)
        assert run.sa(rest, layers, own) == want, (rest, layers, own)
        joined += want
    assert 100 < joined < 300

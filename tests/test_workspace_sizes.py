"""The sizes that the workspace queries report suffice for every call with sizes up to the queried ones (no GPU needed).

What a call asks for is read from its refusal of an empty workspace, which it reports before anything is launched."""
import ctypes as C
import itertools
import random
import re

import pytest

import paper_2410_03804_amd as moa
from paper_2410_03804_amd import binding

LIB = binding._lib
FAKE = 256                                        # a device address that nothing looks at
NO_WS = -6                                        # MOA_ERR_WORKSPACE
SHAPES = {
    "8b": moa.Shape(32, 4096, 32, 8, 128, 2048, 16, 8, moa.BF16),
    "70b": moa.Shape(80, 8192, 64, 8, 128, 2048, 16, 8, moa.BF16),
    "dh64": moa.Shape(8, 1024, 16, 4, 64, 512, 8, 4, moa.BF16),
    "mha": moa.Shape(32, 2048, 16, 16, 128, 2048, 16, 8, moa.BF16),
    "fp32": moa.Shape(4, 256, 4, 2, 64, 256, 4, 2, moa.F32),
}


def need(rc):
    assert rc == NO_WS, (rc, moa.last_error())
    return int(re.search(r"workspace 0 bytes, (\d+) needed", moa.last_error()).group(1))


def ca_need(s, B, Mq, P):
    return need(LIB.moa_cross_attn_draft(C.byref(s), FAKE, B, Mq, FAKE, FAKE, FAKE, FAKE, FAKE, P, FAKE, None, FAKE, 0, None))


def verify_need(s, B, M, P):
    return need(LIB.moa_tree_verify_attn(C.byref(s), FAKE, B, M, *[FAKE] * 7, P, *[FAKE] * 4, None, FAKE, 0, None))


def sa_need(s, B, M, node0, Mn, P):
    return need(LIB.moa_self_attn_draft(C.byref(s), FAKE, B, M, node0, Mn, *[FAKE] * 7, P, *[FAKE] * 4, None, FAKE, 0, None))


def lsa_need(s, T):
    return need(LIB.moa_lsa(C.byref(s), FAKE, T, *[FAKE] * 5, FAKE, 0, None))


def tli_need(s, cfg, B, M, node0, Mn, P):
    return need(LIB.moa_tli_decoder_layer(C.byref(s), C.byref(cfg), FAKE, B, M, node0, Mn, *[FAKE] * 12, P, *[FAKE] * 5, None,
                                          FAKE, 0, None))


def mlp_need(dtype, R, d, f):
    return need(LIB.moa_mlp_block(dtype, FAKE, FAKE, R, d, f, *[FAKE] * 4, 1e-5, FAKE, FAKE, 0, None))


@pytest.mark.parametrize("name", SHAPES)
def test_a_query_covers_every_level_of_its_tree(name):
    """Drafting goes level by level: one workspace, sized for the tree, serves calls over a few of its nodes."""
    s = SHAPES[name]
    for B, cap, breadth, depth in itertools.product((1, 2, 3, 8, 16), (64, 512, 2048, 8192), (2, 8, 16), (2, 4, 8)):
        M = 1 + breadth * depth
        have = moa.workspace_bytes(s, B, cap, M, 0)
        for Mn in {1, breadth, M}:
            assert ca_need(s, B, Mn, cap) <= have, (name, B, cap, M, Mn)
            assert sa_need(s, B, M, 0, Mn, cap) <= have, (name, B, cap, M, Mn)
        assert verify_need(s, B, M, cap) <= have, (name, B, cap, M)


@pytest.mark.parametrize("name", SHAPES)
def test_a_query_covers_smaller_sizes(name):
    rng = random.Random(7)
    s = SHAPES[name]
    for _ in range(1500):
        B, P, M, T = rng.randint(1, 20), rng.randint(1, 9000), rng.randint(1, 256), rng.choice([0, 0, rng.randint(1, 700), 20000])
        have = moa.workspace_bytes(s, B, P, M, T)
        b, p, m, t = rng.randint(1, B), rng.randint(1, P), rng.randint(1, M), rng.randint(0, T)
        assert moa.workspace_bytes(s, b, p, m, t) <= have, (name, (B, P, M, T), (b, p, m, t))
        assert ca_need(s, b, m, p) <= have and verify_need(s, b, m, p) <= have, (name, (B, P, M, T), (b, p, m))
        if t:
            assert lsa_need(s, t) <= have, (name, (B, P, M, T), t)


@pytest.mark.parametrize("name", ["8b", "70b", "dh64", "mha"])
def test_a_steps_query_covers_its_self_attention_layer(name):
    """That layer has key / value heads of its own."""
    rng = random.Random(11)
    s = SHAPES[name]
    for _ in range(1500):
        B, M, P = rng.randint(1, 16), rng.randint(1, 200), rng.choice([1, 64, 300, 1024, 8192])
        kv = rng.choice([h for h in range(1, s.n_q_heads + 1) if s.n_q_heads % h == 0])
        sa = moa.Shape(s.n_layers, s.d_model, s.n_q_heads, kv, s.head_dim, s.d_lsa_in, s.lsa_q_heads, s.lsa_kv_heads, s.dtype)
        assert sa_need(sa, B, M, 0, M, P) <= moa.workspace_bytes(s, B, P, M, 1), (name, B, M, P, kv)


@pytest.mark.parametrize("name", ["8b", "70b", "dh64", "fp32"])
def test_queries_of_blocks_cover_smaller_sizes(name):
    rng = random.Random(9)
    s = SHAPES[name]
    d = s.d_model
    for _ in range(600):
        B, P, M, f = rng.randint(1, 8), rng.randint(1, 4096), rng.randint(1, 256), rng.choice([d // 8, 7 * d // 4, 7 * d // 2, 11008])
        cfg = moa.DecoderCfg(f, 1e-5, 10000.0)
        have = moa.tli_workspace_bytes(s, cfg, B, P, M)
        b, p, m = rng.randint(1, B), rng.randint(1, P), rng.randint(1, M)
        assert moa.tli_workspace_bytes(s, cfg, b, p, m) <= have, (name, f, (B, P, M), (b, p, m))
        assert tli_need(s, cfg, b, M, M - m, m, p) <= have, (name, f, (B, P, M), (b, p, m))
        R, r = B * M, b * m
        have = moa.mlp_block_workspace_bytes(s.dtype, R, d, f)
        assert moa.mlp_block_workspace_bytes(s.dtype, r, d, f) <= have and mlp_need(s.dtype, r, d, f) <= have, (name, f, R, r)
        assert moa.linear_workspace_bytes(s.dtype, r, f, d) <= moa.linear_workspace_bytes(s.dtype, R, f, d), (name, f, R, r)

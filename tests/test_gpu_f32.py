"""GPU parity of the single-precision kernels at the edges of their tiles: the projections with few (16 x 16, K split over
the wavefronts) and many (64 x 64) output tiles, also for bf16 shapes no bf16 matrix kernel takes, and the attention core."""
import numpy as np
import pytest
import torch

import moa_inputs as mi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util
    return gpu_util


@pytest.fixture(scope="module")
def moa(G):
    import paper_2410_03804_amd as m
    return m


CASES = [
    ("f32", 1, 4, 1),             # one piece of one row
    ("f32", 17, 20, 17),          # one past a tile in rows, features and K steps
    ("f32", 16, 256, 768),        # whole tiles, one batch of loads per wavefront
    ("f32", 15, 1044, 33),        # several batches, ragged last one
    ("f32", 8, 8192, 64),
    ("f32", 63, 512, 8128),       # 127 tiles of 64 x 64: the last size of the small form
    ("f32", 64, 512, 8192),       # 128 of them: the first of the large one
    ("f32", 513, 36, 1030),       # ragged in rows, features (no vector stores) and K
    ("f32", 700, 512, 1028),
    ("bf16", 5, 132, 50),
    ("bf16", 600, 260, 1004),
]


@pytest.mark.parametrize("dtype,R,K,N", CASES)
def test_linear_f32_parity(G, moa, oracle, dtype, R, K, N):
    rng = np.random.default_rng(R + 3 * K + N)
    x = mi.quantize(rng.standard_normal((R, K)).astype(np.float32), dtype)
    w = mi.quantize((rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32), dtype)
    print(f"[case] linear {dtype} R={R} K={K} N={N}", flush=True)
    y = torch.full((R, N), float("nan"), dtype=G.TDT[dtype], device="cuda")
    moa.linear(G.dev(x, dtype), G.dev(w, dtype), y)
    torch.cuda.synchronize()
    # sums of K products of order 1/sqrt(K): the rounding of one fp32 sum (bf16: of the result) and its growth over K
    G.check_close(G.host(y), oracle.linear(x, w), dtype, f"linear[{dtype} {R}x{K}x{N}]", residual_stream=True)


@pytest.mark.parametrize("M,H,Hkv,dh,plen", [(7, 6, 2, 128, [129, 0, 16]), (16, 1, 1, 64, [15]), (33, 4, 4, 64, [1, 300]),
                                             (1, 16, 1, 128, [17])])
def test_attn_f32_parity(G, moa, oracle, M, H, Hkv, dh, plen):
    """Query rows that do and do not fill tiles of 16, key ranges around the tiles of 16 and the eight wavefronts, an empty
    prefix, trees of one and of several tiles."""
    cfg = mi.Config(name="f32", index=11, dtype="f32", B=len(plen), P_min=1, P_max=max(plen), M=M, D=min(3, M - 1), max_branch=16, L=2,
                    d=H * dh, H=H, Hkv=Hkv, dh=dh, d_lsa_in=dh, rms_norm=False)
    plen = np.array(plen, dtype=np.int32)
    P_cap = int(plen.max()) + 3
    w, x = mi.verify_weights(cfg), mi.verify_inputs(cfg)
    kc, vc = mi.kv_cache(cfg, which=0, P_cap=P_cap)
    mask_np, _ = oracle.tree_build(mi.trees(cfg))
    print(f"[case] tree_verify f32 M={M} H={H}/{Hkv} dh={dh} len={list(plen)}", flush=True)
    shape = G.shape_of(cfg)
    out = torch.full((cfg.B, M, cfg.d), float("nan"), dtype=torch.float32, device="cuda")
    kt = torch.empty((cfg.B, Hkv, M, dh), dtype=torch.float32, device="cuda")
    vt, st = torch.empty_like(kt), G.status_word()
    moa.tree_verify_attn(shape, G.dev(x), *(G.dev(w[k]) for k in ("wq", "wk", "wv", "wo")), G.dev(kc), G.dev(vc), G.dev(plen), P_cap,
                         G.dev(mask_np.view(np.int64)), out, kt, vt, G.workspace(shape, cfg.B, P_cap, M, 0), st)
    torch.cuda.synchronize()
    want, wkt, _ = oracle.tree_verify_attn(x, w["wq"], w["wk"], w["wv"], w["wo"], kc, vc, plen, mask_np, H, Hkv, dh)
    G.check_close(G.host(kt), wkt, "f32", "k_tree")
    G.check_close(G.host(out), want, "f32", "tree_verify")
    assert st.item() == 0

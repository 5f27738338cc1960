"""GPU parity of the wrappers of the drafter's own layers (moa_rmsnorm, moa_mlp_block) against the fp64 oracle, at the
sizes of the appendix architecture table and on ragged small ones, and of a whole drafter pass composed from the
entry points: embeddings -> [norm, Self-Attention, MLP 512] -> [norm, Cross-Attention over the memory, MLP 7168], with
the memory = MLP-6144 block on the Layer Self-Attention's output."""
import numpy as np
import pytest
import torch

import moa_inputs as mi

pytestmark = pytest.mark.gpu

EPS = 1e-5


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


def block_inputs(dtype, R, d, d_ff, seed, with_res):
    rng = np.random.default_rng(seed)
    x = mi.quantize(rng.standard_normal((R, d)).astype(np.float32), dtype)
    res = mi.quantize((0.5 * rng.standard_normal((R, d))).astype(np.float32), dtype) if with_res else None
    w = dict(g=mi.quantize((1.0 + 0.1 * rng.standard_normal(d)).astype(np.float32), dtype),
             w_gate=mi.quantize((rng.standard_normal((d_ff, d)) / np.sqrt(d)).astype(np.float32), dtype),
             w_up=mi.quantize((rng.standard_normal((d_ff, d)) / np.sqrt(d)).astype(np.float32), dtype),
             w_down=mi.quantize((rng.standard_normal((d, d_ff)) / np.sqrt(d_ff)).astype(np.float32), dtype))
    return x, res, w


def gpu_block(G, moa, dtype, x, res, w, out=None):
    d, d_ff = x.shape[-1], w["w_gate"].shape[0]
    R = x.size // d
    ws = torch.empty(max(moa.mlp_block_workspace_bytes(G.MDT[dtype], R, d, d_ff), 256), dtype=torch.uint8, device="cuda")
    xd = G.dev(x, dtype)
    out = torch.full_like(xd, float("nan")) if out is None else out
    moa.mlp_block(G.MDT[dtype], xd, G.dev(res, dtype), *(G.dev(w[k], dtype) for k in ("g", "w_gate", "w_up", "w_down")),
                  EPS, out, ws)
    torch.cuda.synchronize()
    return out


# (dtype, rows, stream width, MLP size, residual input): the three MLPs of the appendix table on a 60-node tree, the
# same on 130 and 300 rows (other projection kernels), and sizes no fast kernel takes
CASES = [("bf16", 60, 2048, 6144, False), ("bf16", 60, 4096, 512, True), ("bf16", 60, 4096, 7168, True),
         ("bf16", 130, 4096, 512, True), ("bf16", 300, 2048, 6144, False), ("bf16", 8, 4096, 7168, True),
         ("bf16", 19, 192, 320, True), ("bf16", 5, 96, 100, False), ("f32", 19, 192, 320, True), ("f32", 3, 50, 70, False),
         ("f32", 1, 256, 32, True)]


@pytest.mark.parametrize("dtype,R,d,d_ff,with_res", CASES)
def test_mlp_block_parity(G, moa, oracle, dtype, R, d, d_ff, with_res):
    x, res, w = block_inputs(dtype, R, d, d_ff, R + d_ff, with_res)
    print(f"[case] mlp_block {dtype} R={R} d={d} d_ff={d_ff} res={with_res}", flush=True)
    got = gpu_block(G, moa, dtype, x, res, w)
    want = oracle.mlp_block(x, res, w["g"], w["w_gate"], w["w_up"], w["w_down"], EPS)
    G.check_close(G.host(got), want, dtype, f"mlp_block[{dtype} {R}x{d}x{d_ff}]", residual_stream=True)


@pytest.mark.parametrize("dtype,R,d", [("bf16", 60, 4096), ("bf16", 7, 2048), ("bf16", 3, 100), ("f32", 19, 192), ("f32", 2, 7)])
def test_rmsnorm_parity(G, moa, oracle, dtype, R, d):
    rng = np.random.default_rng(R * d)
    x = mi.quantize((3.0 * rng.standard_normal((R, d))).astype(np.float32), dtype)
    g = mi.quantize((1.0 + 0.1 * rng.standard_normal(d)).astype(np.float32), dtype)
    out = torch.full((R, d), float("nan"), dtype=G.TDT[dtype], device="cuda")
    moa.rmsnorm(G.MDT[dtype], G.dev(x, dtype), G.dev(g, dtype), EPS, out)
    torch.cuda.synchronize()
    G.check_close(G.host(out), oracle.rmsnorm(x, g, EPS), dtype, f"rmsnorm[{dtype} {R}x{d}]", residual_stream=True)


def test_mlp_block_in_place_and_empty(G, moa, oracle):
    x, res, w = block_inputs("bf16", 60, 512, 768, 3, True)
    xd = G.dev(x, "bf16")
    ws = torch.empty(moa.mlp_block_workspace_bytes(moa.BF16, 60, 512, 768), dtype=torch.uint8, device="cuda")
    wd = [G.dev(w[k], "bf16") for k in ("g", "w_gate", "w_up", "w_down")]
    moa.mlp_block(moa.BF16, xd, G.dev(res, "bf16"), *wd, EPS, xd, ws)               # out aliases x
    torch.cuda.synchronize()
    want = oracle.mlp_block(x, res, w["g"], w["w_gate"], w["w_up"], w["w_down"], EPS)
    G.check_close(G.host(xd), want, "bf16", "mlp_block[in place]", residual_stream=True)
    empty = torch.empty((0, 512), dtype=torch.bfloat16, device="cuda")
    moa.mlp_block(moa.BF16, empty, None, *wd, EPS, empty, None)                    # nothing to do, nothing needed
    assert moa.mlp_block_workspace_bytes(moa.BF16, 0, 512, 768) >= 0


@pytest.mark.parametrize("R", [60, 240])
def test_mlp_block_output_off_alignment(G, moa, R):
    """An output row that starts off a 16-byte boundary gets the bits an aligned one gets."""
    x, res, w = block_inputs("bf16", R, 512, 768, R, True)
    wd = [G.dev(w[k], "bf16") for k in ("g", "w_gate", "w_up", "w_down")]
    ws = torch.empty(moa.mlp_block_workspace_bytes(moa.BF16, R, 512, 768), dtype=torch.uint8, device="cuda")
    xd, rd = G.dev(x, "bf16"), G.dev(res, "bf16")
    want = torch.empty_like(xd)
    flat = torch.full((R * 512 + 16,), -7.0, dtype=torch.bfloat16, device="cuda")
    got = flat[1:1 + R * 512].view(R, 512)
    print(f"[case] mlp_block R={R} out + 2 bytes", flush=True)
    moa.mlp_block(moa.BF16, xd, rd, *wd, EPS, want, ws)
    moa.mlp_block(moa.BF16, xd, rd, *wd, EPS, got, ws)
    assert torch.equal(got, want)
    assert flat[0] == -7.0 and (flat[1 + R * 512:] == -7.0).all()


def test_block_entry_points_reject_bad_arguments(G, moa):
    x, res, w = block_inputs("bf16", 4, 256, 512, 1, False)
    xd = G.dev(x, "bf16")
    wd = [G.dev(w[k], "bf16") for k in ("g", "w_gate", "w_up", "w_down")]
    out = torch.zeros_like(xd)
    ws = torch.empty(moa.mlp_block_workspace_bytes(moa.BF16, 4, 256, 512), dtype=torch.uint8, device="cuda")
    with pytest.raises(moa.MoaError):
        moa.mlp_block(moa.BF16, xd, None, *wd, EPS, out, ws[:-256])                 # workspace short
    with pytest.raises(moa.MoaError):
        moa.mlp_block(moa.BF16, xd, None, *wd, -1.0, out, ws)                       # negative epsilon
    with pytest.raises((moa.MoaError, KeyError)):
        moa.mlp_block(7, xd, None, *wd, EPS, out, ws)                               # no such dtype
    with pytest.raises(moa.MoaError):
        moa.rmsnorm(moa.BF16, xd, wd[0], float("nan"), out)
    torch.cuda.synchronize()
    assert torch.count_nonzero(out).item() == 0                                     # nothing was launched


def drafter_cfg(dtype):
    return mi.Config(name="DRAFTER", index=19, dtype=dtype, B=2, P_min=30, P_max=180, M=23, D=4, max_branch=4, L=3, d=512,
                     H=8, Hkv=4, dh=64, d_lsa_in=256, rms_norm=True)


@pytest.mark.parametrize("case", ["small_f32", "small_bf16", "C1_bf16"])
def test_drafter_pass_composed_from_the_entry_points(G, moa, oracle, case):
    """One pass of the drafter's own layers on a whole tree, every sub-layer wrapped: the memory rows come from
    LSA -> MLP block, the queries from the Self-Attention layer, the output from the Cross-Attention layer."""
    cfg = {"small_f32": drafter_cfg("f32"), "small_bf16": drafter_cfg("bf16"), "C1_bf16": mi.CONFIGS["C1"]}[case]
    dt, mdt, tdt = cfg.dtype, G.MDT[cfg.dtype], G.TDT[cfg.dtype]
    B, M, d, dh = cfg.B, cfg.M, cfg.d, cfg.dh
    T = 2 * B                                                       # two newly verified tokens per sequence join the memory
    print(f"[case] drafter pass {case} B={B} M={M} d={d} T={T}", flush=True)
    hkv_sa = mi.sa_kv_heads(cfg)
    lsa_w, ca_w, sa_w = mi.lsa_weights(cfg), mi.ca_weights(cfg), mi.sa_weights(cfg)
    mlp = {k: mi.drafter_mlp_weights(cfg, k) for k in ("lsa", "sa", "ca")}
    gain = {k: mi.drafter_norm_gain(cfg, k) for k in ("sa", "ca")}
    hs = mi.lsa_inputs(cfg, T)
    emb, sa_kc, sa_vc = mi.sa_inputs(cfg)
    plen = mi.prefix_lengths(cfg)
    parent = mi.trees(cfg)
    mask_np, _ = oracle.tree_build(parent)
    ca_k0, ca_v0 = mi.kv_cache(cfg, which=3)                         # the memory's projected rows so far
    P_cap = ca_k0.shape[2]
    tok_off = np.arange(0, T + 1, 2, dtype=np.int32)

    # ---- oracle
    a = oracle.lsa(hs, lsa_w["wq"], lsa_w["wk"], lsa_w["wv"], lsa_w["wo"], cfg.lsa_heads, cfg.Hkv, dh)
    mem = oracle.mlp_block(a, None, *(mlp["lsa"][k] for k in ("g", "w_gate", "w_up", "w_down")), EPS)
    mem_q = mi.quantize(mem.astype(np.float32), dt)                  # the library hands the rows on in the storage type
    wk_c, wv_c = ca_k0.astype(np.float64).copy(), ca_v0.astype(np.float64).copy()
    want_len = plen.copy()
    oracle.ca_kv_append(mem_q, tok_off, ca_w["wk"], ca_w["wv"], wk_c, wv_c, want_len, cfg.Hkv, dh)
    n_sa = oracle.rmsnorm(emb, gain["sa"], EPS)
    n_sa_q = mi.quantize(n_sa.astype(np.float32), dt)
    kd = np.zeros((B, hkv_sa, M, dh))
    sa_out = oracle.self_attn_draft(n_sa_q, parent, 0, sa_w["wq"], sa_w["wk"], sa_w["wv"], sa_w["wo"], sa_kc, sa_vc, plen,
                                    kd, kd.copy(), cfg.H, hkv_sa, dh)
    sa_out_q = mi.quantize(sa_out.astype(np.float32), dt)
    q = oracle.mlp_block(emb, sa_out_q, *(mlp["sa"][k] for k in ("g", "w_gate", "w_up", "w_down")), EPS)
    q_q = mi.quantize(q.astype(np.float32), dt)
    n_ca_q = mi.quantize(oracle.rmsnorm(q_q, gain["ca"], EPS).astype(np.float32), dt)
    wk_q, wv_q = mi.quantize(wk_c.astype(np.float32), dt), mi.quantize(wv_c.astype(np.float32), dt)
    ca_out = oracle.cross_attn(n_ca_q, ca_w["wq"], ca_w["wo"], wk_q, wv_q, want_len, cfg.H, cfg.Hkv, dh)
    ca_out_q = mi.quantize(ca_out.astype(np.float32), dt)
    want = oracle.mlp_block(q_q, ca_out_q, *(mlp["ca"][k] for k in ("g", "w_gate", "w_up", "w_down")), EPS)

    # ---- library
    shape = G.shape_of(cfg)
    shape_sa = moa.Shape(cfg.L, d, cfg.H, hkv_sa, dh, cfg.d_lsa_in, cfg.lsa_heads, cfg.Hkv, mdt)
    st = G.status_word()
    ws = G.workspace(shape, B, P_cap, M, T)
    D = lambda arr: G.dev(arr, dt)
    blk_ws = lambda R, dd, ff: torch.empty(max(moa.mlp_block_workspace_bytes(mdt, R, dd, ff), 256), dtype=torch.uint8, device="cuda")
    mw = {k: [D(mlp[k][n]) for n in ("g", "w_gate", "w_up", "w_down")] for k in mlp}
    lsa_out = torch.empty((T, cfg.d_lsa), dtype=tdt, device="cuda")
    moa.lsa(shape, D(hs), *(D(lsa_w[k]) for k in ("wq", "wk", "wv", "wo")), lsa_out, ws)
    mem_d = torch.empty_like(lsa_out)
    moa.mlp_block(mdt, lsa_out, None, *mw["lsa"], EPS, mem_d, blk_ws(T, cfg.d_lsa, mlp["lsa"]["w_gate"].shape[0]))
    kc_d, vc_d, len_d = D(ca_k0), D(ca_v0), G.dev(plen.copy())
    moa.ca_kv_append(shape, mem_d, G.dev(tok_off), D(ca_w["wk"]), D(ca_w["wv"]), kc_d, vc_d, len_d, P_cap, st, ws)
    emb_d = D(emb)
    n_d = torch.empty_like(emb_d)
    moa.rmsnorm(mdt, emb_d, D(gain["sa"]), EPS, n_d)
    sa_d = torch.empty_like(emb_d)
    kdd = torch.zeros((B, hkv_sa, M, dh), dtype=tdt, device="cuda")
    moa.self_attn_draft(shape_sa, n_d, 0, *(D(sa_w[k]) for k in ("wq", "wk", "wv", "wo")), D(sa_kc), D(sa_vc), G.dev(plen),
                        sa_kc.shape[2], G.dev(mask_np.view(np.int64)), sa_d, kdd, torch.zeros_like(kdd), ws, st)
    q_d = torch.empty_like(emb_d)
    moa.mlp_block(mdt, emb_d, sa_d, *mw["sa"], EPS, q_d, blk_ws(B * M, d, mlp["sa"]["w_gate"].shape[0]))
    moa.rmsnorm(mdt, q_d, D(gain["ca"]), EPS, n_d)
    ca_d = torch.empty_like(emb_d)
    moa.cross_attn_draft(shape, n_d, D(ca_w["wq"]), D(ca_w["wo"]), kc_d, vc_d, len_d, P_cap, ca_d, ws, st)
    out_d = torch.empty_like(emb_d)
    moa.mlp_block(mdt, q_d, ca_d, *mw["ca"], EPS, out_d, blk_ws(B * M, d, mlp["ca"]["w_gate"].shape[0]))
    torch.cuda.synchronize()
    assert st.item() == 0
    assert np.array_equal(len_d.cpu().numpy(), want_len)

    # every stage against the oracle's, which took its own previous stage rounded to the storage type (the library's
    # differs from that by the library's rounding error): the output has been through two residual blocks
    G.check_close(G.host(mem_d), mem, dt, f"drafter.memory_rows[{case}]", residual_stream=True)
    G.check_close(G.host(q_d), q, dt, f"drafter.queries[{case}]", residual_stream=True)
    G.check_close(G.host(out_d), want, dt, f"drafter.out[{case}]", residual_stream=True, stages=2)

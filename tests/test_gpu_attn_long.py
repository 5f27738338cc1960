"""GPU parity of the attention kernel for more than 128 query rows per (sequence, KV head) at the edges of its tiles: row
counts around 128 and 256 and in several row tiles, key ranges around the 64-key tiles and the two 32-key halves of one,
an empty prefix, slices of the key range that hold no key, one slice (no merge pass), trees of one to three mask words, and
scores that move the reference of the exponent between tiles."""
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


@pytest.fixture(params=["split_wide", "split"])
def moa(G, request):
    """256-row tiles, then the tiles that the estimate of the time picks (128 rows for most of these small calls)."""
    import paper_2410_03804_amd as m
    m.debug_force_attn_kernel(request.param)
    yield m
    m.debug_force_attn_kernel("auto")


CASES = [
    # M, H, Hkv, prefix lengths, cache rows per sequence, factor on the queries
    (43, 3, 1, [0, 1, 31, 64], 70, 1.0),             # 129 rows: one 256-row tile, half of it empty
    (64, 4, 1, [65, 128, 129], 400, 1.0),            # 256 rows exactly; slices without a key
    (65, 4, 1, [191, 33], 1024, 1.0),                # 260 rows: two row tiles, a tree of two tiles
    (130, 2, 1, [300, 97], 640, 4.0),                # a tree of three tiles, peaked scores
    (173, 6, 2, [5, 1000], 2100, 1.0),               # 519 rows: three row tiles, two KV heads
    (130, 4, 2, [257] * 32, 260, 1.0),               # 64 (sequence, head) pairs of two row tiles: two slices
    (65, 64, 16, [40] * 16, 100, 1.0),               # 256 pairs of two row tiles: one slice, no merge pass
    (70, 8, 2, [999], 1000, 30.0),                   # scores of order 100: the reference moves at most tiles
]


@pytest.mark.parametrize("M,H,Hkv,plen,P_cap,factor", CASES)
def test_attn_long_tile_edges(G, moa, oracle, M, H, Hkv, plen, P_cap, factor):
    cfg = mi.Config(name="long", index=13, dtype="bf16", B=len(plen), P_min=1, P_max=max(max(plen), 1), M=M, D=7, max_branch=5, L=2,
                    d=256, H=H, Hkv=Hkv, dh=128, d_lsa_in=256, rms_norm=True)
    plen = np.array(plen, dtype=np.int32)
    w, x = mi.verify_weights(cfg), mi.verify_inputs(cfg)
    w["wq"] = mi.quantize(w["wq"] * factor, "bf16")
    kc, vc = mi.kv_cache(cfg, which=0, P_cap=P_cap)
    for b, n in enumerate(plen):                     # rows past a sequence's length are never used
        kc[b, :, n:], vc[b, :, n:] = np.nan, np.nan
    mask_np, _ = oracle.tree_build(mi.trees(cfg))
    print(f"[case] tree_verify M={M} H={H}/{Hkv} B={cfg.B} P_cap={P_cap} factor={factor}", flush=True)
    shape = G.shape_of(cfg)
    out = torch.full((cfg.B, M, cfg.d), float("nan"), dtype=torch.bfloat16, device="cuda")
    kt = torch.empty((cfg.B, Hkv, M, 128), dtype=torch.bfloat16, device="cuda")
    vt, st = torch.empty_like(kt), G.status_word()
    moa.tree_verify_attn(shape, G.dev(x, "bf16"), *(G.dev(w[k], "bf16") for k in ("wq", "wk", "wv", "wo")), G.dev(kc, "bf16"),
                         G.dev(vc, "bf16"), G.dev(plen), P_cap, G.dev(mask_np.view(np.int64)), out, kt, vt,
                         G.workspace(shape, cfg.B, P_cap, M, 0), st)
    torch.cuda.synchronize()
    assert st.item() == 0
    want, _, _ = oracle.tree_verify_attn(x, w["wq"], w["wk"], w["wv"], w["wo"], kc, vc, plen, mask_np, H, Hkv, 128)
    if factor == 1.0:
        G.check_close(G.host(out), want, "bf16", f"tree_verify[{M}x{H}/{Hkv}]")
        return
    # queries of size `factor` are rounded to 2^-9 of that, so a score is off by up to factor * 2^-9 rms and a weight by as much
    # relative to itself; 2^-8 for the roundings of the rest.  The largest element of 10^5 at six times the rms
    got = G.host(out)
    assert np.all(np.isfinite(got))
    bound = factor * 2.0 ** -9 + 2.0 ** -8
    assert np.linalg.norm(got - want) <= bound * np.linalg.norm(want)
    assert np.abs(got - want).max() <= 6 * bound * np.sqrt(np.mean(want ** 2))


@pytest.mark.parametrize("M,kernel", [(65, "k_attn_mfma<128, 1>"), (96, "k_attn_mfma<128, 1>"), (97, "k_attn_long<128>"),
                                      (128, "k_attn_long<128>")])
def test_row_tile_height_follows_how_well_rows_fill_it(G, M, kernel):
    """8 sequences x 8 KV heads: up to 384 rows three tiles of 128 keep the chip busy where two of 256 leave half of it idle
    (their scratch would not hold two key slices); from there on 256-row tiles are the faster ones."""
    import paper_2410_03804_amd as m
    B, P = 8, 4096
    shape = m.Shape(2, 4096, 32, 8, 128, 256, 2, 1, m.BF16)
    print(f"[case] cross_attn_draft B={B} M={M} P_cap={P}", flush=True)
    kc, x = torch.randn(B, 8, P, 128, device="cuda").bfloat16(), torch.randn(B, M, 4096, device="cuda").bfloat16()
    out, ln = torch.empty_like(x), torch.full((B,), P, dtype=torch.int32, device="cuda")
    ws = torch.empty(m.workspace_bytes(shape, B, P, M, 0), dtype=torch.uint8, device="cuda")
    names = G.kernels_of(lambda: m.cross_attn_draft(shape, x, None, None, kc, kc, ln, P, out, ws, G.status_word()))
    assert kernel in names, names


@pytest.mark.parametrize("factor", [1.0, 3.0, 8.0])
def test_wide_row_tiles_round_the_weights_no_worse(G, factor):
    """The 256-row form against 64 bits, beside the whole-key-range form: both take the running maximum as the exponent's
    reference, so the heaviest weights lose least when they are rounded to bf16.  A reference that lags behind gives 1.04
    (flat weights) to 1.2 times the error (peaked ones); the forms differ by a few percent of a tenth of it in the order of
    their sums and the rounding of partial results to fp16 (2^-12 against 2^-9)."""
    import paper_2410_03804_amd as m
    B, M, H, Hkv, P = 1, 64, 16, 4, 4096                        # 256 rows per KV head
    g = torch.Generator(device="cuda").manual_seed(3)
    shape = m.Shape(2, H * 128, H, Hkv, 128, 256, 2, 1, m.BF16)
    q = (torch.randn(B, M, H * 128, generator=g, device="cuda") * factor).bfloat16()
    k, v = (torch.randn(B, Hkv, P, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    ln = torch.full((B,), P, dtype=torch.int32, device="cuda")
    heads = q[0].view(M, Hkv, H // Hkv, 128).permute(1, 0, 2, 3).reshape(Hkv, -1, 128).double().cpu()
    want = torch.stack([torch.softmax(heads[i] @ k[0, i].double().cpu().T / 128 ** 0.5, -1) @ v[0, i].double().cpu() for i in range(Hkv)])
    err = {}
    for form in ("whole", "split_wide"):
        print(f"[case] cross_attn_draft {form} factor={factor}", flush=True)
        m.debug_force_attn_kernel(form)
        try:
            out = torch.empty_like(q)
            ws = torch.empty(m.workspace_bytes(shape, B, P, M, 0), dtype=torch.uint8, device="cuda")
            m.cross_attn_draft(shape, q, None, None, k, v, ln, P, out, ws, G.status_word())
            torch.cuda.synchronize()
        finally:
            m.debug_force_attn_kernel("auto")
        got = out[0].view(M, Hkv, H // Hkv, 128).permute(1, 0, 2, 3).reshape(Hkv, -1, 128).double().cpu()
        err[form] = ((got - want).norm() / want.norm()).item()
    print(err)
    assert err["split_wide"] <= 1.02 * err["whole"], err


@pytest.mark.parametrize("M,H,factor", [(33, 32, 1.0), (64, 32, 6.0)])
def test_rounds_of_three_full_tiles_and_what_follows_them(G, moa, request, M, H, factor):
    """Slices of 2 .. 13 tiles of 64 keys, ending on, before and behind a tile: rounds of three unmasked tiles, their one to five
    masked followers and slices that have only those.  Against 64 bits; weights and result are rounded to bf16 (2^-9 each) and a
    slice's result to fp16, a largest element of 10^6 at six times that."""
    B, Hkv, P = 16, 8, 1600
    lens = [255, 256, 257, 383, 384, 447, 448, 511, 513, 640, 769, 896, 1023, 1280, 1537, 1600]
    g = torch.Generator(device="cuda").manual_seed(5)
    shape = moa.Shape(2, H * 128, H, Hkv, 128, 256, 2, 1, moa.BF16)
    q = (torch.randn(B, M, H * 128, generator=g, device="cuda") * factor).bfloat16()
    k, v = (torch.randn(B, Hkv, P, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    for b, n in enumerate(lens):                                # rows past a sequence's length are never used
        k[b, :, n:], v[b, :, n:] = float("nan"), float("nan")
    print(f"[case] cross_attn_draft M={M} factor={factor}", flush=True)
    out = torch.empty_like(q)
    ws = torch.empty(moa.workspace_bytes(shape, B, P, M, 0), dtype=torch.uint8, device="cuda")
    plen = torch.tensor(lens, dtype=torch.int32, device="cuda")
    names = G.kernels_of(lambda: moa.cross_attn_draft(shape, q, None, None, k, v, plen, P, out, ws, G.status_word()))
    assert request.node.callspec.params["moa"] != "split_wide" or "k_attn_long<128>" in names, names
    for b, n in enumerate(lens):
        qb = q[b].view(M, Hkv, H // Hkv, 128).permute(1, 0, 2, 3).reshape(Hkv, -1, 128).double().cpu()
        got = out[b].view(M, Hkv, H // Hkv, 128).permute(1, 0, 2, 3).reshape(Hkv, -1, 128).double().cpu()
        for h in range(Hkv):
            want = torch.softmax(qb[h] @ k[b, h, :n].double().cpu().T / 128 ** 0.5, -1) @ v[b, h, :n].double().cpu()
            diff, rms = got[h] - want, want.square().mean().sqrt()
            assert diff.square().mean().sqrt() <= 2.0 ** -8 * rms, (b, h)
            assert diff.abs().max() <= 6 * 2.0 ** -8 * max(rms, want.abs().max() / 4), (b, h)

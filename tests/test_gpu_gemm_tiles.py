"""GPU parity of the bf16 projection kernel at the edges of its tiles: row counts around each tile height, feature counts
that leave part of the last tile empty, fewer k tiles than the load rings have stages, K cut into slices, and the gated
activation and the residual applied inside the kernel (moa_mlp_block) on ragged sizes."""
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
    (1, 128, 32),            # two k tiles, fewer than any ring's stages
    (32, 256, 4128),         # 32-row tiles, ragged last feature tile
    (7, 384, 16416),         # K groups of two only, many tiles
    (16, 512, 20000),        # four K groups (K in 256s), two workgroups per compute unit
    (32, 640, 31904),        # pairs of feature blocks, half a tile at the end
    (33, 128, 4096),
    (64, 1152, 10272),       # 64 x 64 tiles, half a tile at the end
    (61, 2048, 28704),       # 64 x 128
    (65, 384, 8192),
    (64, 12288, 2048),       # K in slices
    (129, 12288, 1024),      # the same, three 64-row pieces
    (192, 640, 4128),
    (193, 256, 8224),
    (300, 896, 6176),
    (257, 1024, 18464),      # two row tiles of 256, one row in the second
    (1000, 640, 10272),      # 256-row tiles, ragged everywhere
    (2049, 512, 8224),
]


@pytest.mark.parametrize("R,K,N", CASES)
def test_gemm_tile_edges(G, moa, R, K, N):
    print(f"[case] linear bf16 R={R} K={K} N={N}", flush=True)
    g = torch.Generator().manual_seed(R + K + N)
    x = torch.randn(R, K, generator=g).bfloat16()
    w = (torch.randn(N, K, generator=g) / K ** 0.5).bfloat16()
    y = torch.full((R + 1, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(max(moa.linear_workspace_bytes(moa.BF16, R, K, N), 256), dtype=torch.uint8, device="cuda")
    moa.linear(x.cuda(), w.cuda(), y[:R], ws)
    torch.cuda.synchronize()
    assert torch.isnan(y[R]).all(), "rows past the end are not written"
    # fp32 on the GPU by the library routine: sums of K exact products, error K eps of order-1 results; one bf16 rounding
    # of a value up to 5 sigma (2^-9 of it = 1e-2) bounds the difference, and its rms is 2^-9 / sqrt(3)
    want = x.cuda().float() @ w.cuda().float().t()
    diff = (y[:R].float() - want).abs()
    assert diff.max().item() <= 2.0 ** -8 * want.abs().max().item()
    assert (diff.norm() / want.norm()).item() <= 2.0 ** -9


@pytest.mark.parametrize("R,K,N", [(1, 4224, 8192), (8, 640, 53024), (32, 256, 131104), (60, 128, 4096), (200, 1152, 30016)])
def test_wide_matrices_at_odd_k_tile_counts(G, moa, R, K, N):
    """64 MB of weights at a few row counts, and narrower ones: k tile counts that eight does not divide (66, 33, 18), fewer
    than eight (5, 2) and one per K group (60 rows x 128)."""
    print(f"[case] linear bf16 R={R} K={K} N={N}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(R + K)
    x = torch.randn(R, K, generator=g, device="cuda").bfloat16()
    w = (torch.randn(N, K, generator=g, device="cuda") / K ** 0.5).bfloat16()
    y = torch.full((R, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    moa.linear(x, w, y, torch.empty(max(moa.linear_workspace_bytes(moa.BF16, R, K, N), 256), dtype=torch.uint8, device="cuda"))
    want = x.float() @ w.float().t()                          # bounds as in test_gemm_tile_edges
    diff = (y.float() - want).abs()
    assert diff.max().item() <= 2.0 ** -8 * want.abs().max().item()
    assert (diff.norm() / want.norm()).item() <= 2.0 ** -9


@pytest.mark.parametrize("R,K,N,period", [(8, 4096, 128256, 4096), (1, 4096, 32000, 2048), (60, 4096, 28672, 1024), (60, 4096, 4160, 128),
                                          (96, 2048, 8192, 512), (200, 4096, 8224, 512), (64, 14336, 4096, 256)])
def test_equal_weight_rows_give_equal_logits(G, moa, R, K, N, period):
    """The order of a sum along K does not depend on where its feature lies: rows that stand once in every XCD's share of the matrix
    give the same bits everywhere, so that tied tokens stay tied and the most probable ones are the lowest ids.  (Another
    order moves about one sum in two thousand to the next bf16 number: there are 2000 .. 200000 pairs here.)"""
    print(f"[case] linear + topk_logprob R={R} K={K} N={N}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(R + K + N)
    x = torch.randn(R, K, generator=g, device="cuda").bfloat16()
    rows = (torch.randn(period, K, generator=g, device="cuda") / K ** 0.5).bfloat16()
    w = rows.repeat(N // period + 1, 1)[:N].contiguous()
    y = torch.full((R, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    moa.linear(x, w, y, torch.empty(max(moa.linear_workspace_bytes(moa.BF16, R, K, N), 256), dtype=torch.uint8, device="cuda"))
    tok, logp = torch.full((R, 8), -1, dtype=torch.int32, device="cuda"), torch.empty(R, 8, device="cuda")
    moa.topk_logprob(y, 8, tok, logp, torch.empty(max(moa.topk_workspace_bytes(R, N, 8), 256), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert torch.isfinite(y).all()
    assert (y != y[:, :period].repeat(1, N // period + 1)[:, :N]).sum().item() == 0
    for r in range(R):                                       # ids in the order of falling logits, ties by rising id
        ids = torch.sort(y[r].float(), descending=True, stable=True).indices[:8].int()
        assert torch.equal(tok[r], ids), (r, tok[r].tolist(), ids.tolist())


@pytest.mark.parametrize("M", [32, 60, 128])
def test_equal_weight_rows_give_equal_outputs_in_the_layers(G, moa, M):
    """The same for the projections whose sums a step's schedules have to agree on (pairs of K groups and single chains):
    equal rows of W_o give equal features."""
    print(f"[case] cross_attn_draft M={M}", flush=True)
    H, Hkv, d = 32, 8, 4096
    g = torch.Generator(device="cuda").manual_seed(M)
    shape = moa.Shape(2, d, H, Hkv, 128, 256, 2, 1, moa.BF16)
    x = torch.randn(1, M, d, generator=g, device="cuda").bfloat16()
    wq = (torch.randn(H * 128, d, generator=g, device="cuda") / d ** 0.5).bfloat16()
    wo = (torch.randn(256, H * 128, generator=g, device="cuda") / d ** 0.5).bfloat16().repeat(d // 256, 1).contiguous()
    k, v = (torch.randn(1, Hkv, 64, 128, generator=g, device="cuda").bfloat16() for _ in range(2))
    out = torch.full_like(x, float("nan"))
    moa.cross_attn_draft(shape, x, wq, wo, k, v, torch.tensor([64], dtype=torch.int32, device="cuda"), 64, out,
                         G.workspace(shape, 1, 64, M, 0), G.status_word())
    torch.cuda.synchronize()
    assert torch.isfinite(out).all()
    assert (out != out[..., :256].repeat(1, 1, d // 256)).sum().item() == 0


@pytest.mark.parametrize("R,K,N", [(64, 14336, 4096), (129, 12288, 1024)])
def test_without_a_workspace_the_plan_is_made_for_whole_k(G, moa, R, K, N):
    """The tile that is best for several K slices leaves most of the chip idle when there is no room for their sums: without
    a workspace another kernel runs, with the same result."""
    g = torch.Generator().manual_seed(R)
    x, w = torch.randn(R, K, generator=g).bfloat16().cuda(), (torch.randn(N, K, generator=g) / K ** 0.5).bfloat16().cuda()
    ws = torch.empty(moa.linear_workspace_bytes(moa.BF16, R, K, N), dtype=torch.uint8, device="cuda")
    assert ws.numel() > 0                                     # K is cut
    out, kernels = [], []
    for room in (ws, None):
        print(f"[case] linear bf16 R={R} K={K} N={N} workspace={room is not None}", flush=True)
        y = torch.full((R, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        moa.profile_enable(True)
        try:
            moa.linear(x, w, y, room)
            torch.cuda.synchronize()
            kernels.append({k for _, k, _, _ in moa.profile_collect()})
        finally:
            moa.profile_enable(False)
        out.append(y.float())
    assert len(kernels[0]) == 2 and len(kernels[1]) == 1 and not kernels[1] <= kernels[0], kernels
    # each within one bf16 rounding of the product (see above)
    assert (out[0] - out[1]).abs().max().item() <= 2.0 ** -7 * out[0].abs().max().item()


@pytest.mark.parametrize("R,d,d_ff", [(7, 512, 96), (33, 256, 2080), (64, 1024, 7200), (100, 512, 608), (260, 384, 1056)])
def test_mlp_block_ragged_sizes(G, moa, oracle, R, d, d_ff):
    rng = np.random.default_rng(R + d + d_ff)
    q = lambda a: mi.quantize(a.astype(np.float32), "bf16")
    x, res = q(rng.standard_normal((R, d))), q(0.5 * rng.standard_normal((R, d)))
    g = q(1.0 + 0.1 * rng.standard_normal(d))
    wg, wu, wd = (q(rng.standard_normal(s) / np.sqrt(s[1])) for s in ((d_ff, d), (d_ff, d), (d, d_ff)))
    print(f"[case] mlp_block R={R} d={d} d_ff={d_ff}", flush=True)
    out = torch.full((R, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(max(moa.mlp_block_workspace_bytes(moa.BF16, R, d, d_ff), 256), dtype=torch.uint8, device="cuda")
    dev = [G.dev(a, "bf16") for a in (x, res, g, wg, wu, wd)]
    moa.mlp_block(moa.BF16, dev[0], dev[1], *dev[2:], 1e-5, out, ws)
    torch.cuda.synchronize()
    want = oracle.mlp_block(x, res, g, wg, wu, wd, 1e-5)
    G.check_close(G.host(out), want, "bf16", f"mlp_block[{R}x{d}x{d_ff}]", residual_stream=True)


@pytest.mark.parametrize("R,d,V", [(32, 256, 4130), (33, 512, 65600), (64, 128, 300), (65, 256, 66000), (128, 384, 1000), (129, 256, 4099),
                                   (256, 128, 257), (300, 256, 65601), (3, 128, 1)])
def test_lm_head_tiles(G, moa, R, d, V):
    """The LM head's arg-max in each of its tiles, with ragged vocabularies and more rows than one pass takes.  Inputs are
    small integers, so every logit is exact in fp32 whatever the order of the sum: ids (ties to the lower one) and winning
    logits must be exactly those of the fp64 product."""
    print(f"[case] lm_head R={R} d={d} V={V}", flush=True)
    g = torch.Generator().manual_seed(R + d + V)
    x, w = torch.randint(-3, 4, (R, d), generator=g), torch.randint(-3, 4, (V, d), generator=g)
    tgt, best = torch.full((R,), -1, dtype=torch.int32, device="cuda"), torch.zeros(R, device="cuda")
    ws = torch.empty(max(moa.lm_head_workspace_bytes(V), 256), dtype=torch.uint8, device="cuda")
    moa.lm_head_argmax(x.bfloat16().cuda(), w.bfloat16().cuda(), tgt, ws, best)
    torch.cuda.synchronize()
    logits = (x.double() @ w.double().t()).numpy()
    assert np.array_equal(tgt.cpu().numpy(), np.argmax(logits, axis=1))
    assert np.array_equal(best.cpu().numpy().astype(np.float64), logits.max(axis=1))

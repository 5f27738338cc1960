"""The whole-key-range attention in blocks of 16 and of 32 query rows: the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture()
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util
    gpu_util.moa.debug_force_attn_kernel("whole")
    yield gpu_util
    gpu_util.moa.debug_force_attn_kernel("auto")


# (rows per (sequence, KV head) = M H / Hkv; key counts around tiles of 32 and rounds of eight of them.  With as many KV heads as heads
# the tree's keys need no projection, whose sums may depend on the number of rows.)
@pytest.mark.parametrize("M,P", [(1, 1), (3, 31), (4, 32), (5, 33), (15, 64), (16, 255), (17, 257), (37, 300), (60, 1024), (60, 17), (128, 90)])
@pytest.mark.parametrize("H,tree", [(32, False), (8, False), (8, True)], ids=["cross", "cross-g1", "tree"])
def test_both_block_heights_give_the_same_bits(G, M, P, H, tree):
    """One sequence alone takes 16-row blocks; among copies of itself, enough for more than 256 blocks, it takes 32-row ones.  The largest
    has 128 x 4 rows per KV head: 256 blocks of 16."""
    moa = G.moa
    print(f"[case] attention M={M} P={P} H={H} tree={tree}", flush=True)
    Hkv, dh = 8, 128
    shape = moa.Shape(2, H * dh, H, Hkv, dh, 256, 2, 1, moa.BF16)
    g = torch.Generator(device="cuda").manual_seed(M + P)
    rn = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    q, k, v = rn(1, M, H * dh), rn(1, Hkv, P, dh), rn(1, Hkv, P, dh)
    mask = torch.randint(-2**62, 2**62, (1, M, (M + 63) // 64), generator=g, device="cuda")
    mask[:, M // 2] = 0                                    # a row that sees the cache alone
    length = torch.tensor([max(0, P - 3)], dtype=torch.int32, device="cuda")
    outs = []
    for B in (1, 40):
        rep = lambda t: t.expand(B, *t.shape[1:]).contiguous()
        out = torch.full((B, M, H * dh), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = torch.empty(moa.workspace_bytes(shape, B, P, M, 0), dtype=torch.uint8, device="cuda")
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        lens = rep(length[None])[:, 0].contiguous()
        kt, vt = (torch.zeros(B, Hkv, M, dh, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        names = G.kernels_of(lambda: moa.tree_verify_attn(shape, rep(q), None, None, None, None, rep(k), rep(v), lens, P, rep(mask), out, kt, vt, ws, status) if tree
                             else moa.cross_attn_draft(shape, rep(q), None, None, rep(k), rep(v), lens, P, out, ws, status))
        assert [n for n in names if "attn" in n] == ["k_attn_fused16<128, 8>" if B == 1 else "k_attn_fused<128, 8>"], names
        outs.append(out)
    assert torch.isfinite(outs[0].float()).all()
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[1][:1].expand_as(outs[1]), outs[1])

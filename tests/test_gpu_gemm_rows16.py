"""bf16 projections and the LM head around 16 rows, where the tiles change height."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def moa():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2410_03804_amd as m
    return m


def operands(R, K, N):
    g = torch.Generator(device="cuda").manual_seed(R + K + N)
    return (torch.randn(R, K, generator=g, device="cuda").bfloat16(), (torch.randn(N, K, generator=g, device="cuda") / K ** 0.5).bfloat16())


@pytest.mark.parametrize("R", [1, 15, 16, 17, 31])
@pytest.mark.parametrize("K,N", [(128, 32), (1024, 4096), (4096, 4128), (384, 16416), (512, 20000), (640, 31904), (256, 131104), (12288, 1024)])
def test_projection_rows(moa, R, K, N):
    print(f"[case] linear bf16 R={R} K={K} N={N}", flush=True)
    x, w = operands(R, K, N)
    y = torch.full((R + 1, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(max(moa.linear_workspace_bytes(moa.BF16, R, K, N), 256), dtype=torch.uint8, device="cuda")
    moa.linear(x, w, y[:R], ws)
    want = x.float() @ w.float().t()
    torch.cuda.synchronize()
    assert torch.isnan(y[R]).all(), "rows past the end are not written"
    # exact products summed in fp32 on both sides (each sum within K eps of the sum of their magnitudes), then one rounding to
    # eight significant bits: at most 2^-8 of the value
    eps_sum = 2 * K * 2.0 ** -24 * (x.float().abs() @ w.float().abs().t())
    assert ((y[:R].float() - want).abs() <= 2.0 ** -8 * want.abs() + eps_sum).all()


@pytest.mark.parametrize("K,N", [(128, 32), (2048, 2048), (4096, 1024), (4096, 4096), (4096, 6144), (8192, 8192), (14336, 4096), (4096, 28672), (1024, 131104)])
def test_a_rows_sums_do_not_depend_on_the_rows_beside_it(moa, K, N):
    """Up to 32 rows, in tiles of 16 rows and of 32: the same bits (without a workspace, whose slices of K are fewer for more rows)."""
    print(f"[case] linear bf16 1, 8, 16, 17 of 32 rows K={K} N={N}", flush=True)
    x, w = operands(32, K, N)
    ys = []
    for R in (32, 1, 8, 16, 17):
        y = torch.full((R, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        moa.linear(x[:R].contiguous(), w, y, None)
        ys.append(y)
    torch.cuda.synchronize()
    for y in ys[1:]:
        assert torch.equal(y, ys[0][:y.shape[0]]), f"{y.shape[0]} rows"


@pytest.mark.parametrize("R", [1, 16, 17, 32])
def test_head_rows(moa, R, K=256, V=3001):
    print(f"[case] lm_head R={R} K={K} V={V}", flush=True)
    x, w = operands(R, K, V)
    tgt, best = torch.zeros(R, dtype=torch.int32, device="cuda"), torch.zeros(R, device="cuda")
    moa.lm_head_argmax(x, w, tgt, torch.empty(moa.lm_head_workspace_bytes(V), dtype=torch.uint8, device="cuda"), best=best)
    want = x.double() @ w.double().t()
    torch.cuda.synchronize()
    top = want.max(1).values
    # fp32 sums of 256 exact products of order-1 results: 256 eps
    assert (want.gather(1, tgt.long()[:, None])[:, 0] >= top - 256 * 2.0 ** -24 * 4).all()
    assert ((best.double() - top).abs() <= 256 * 2.0 ** -24 * 4).all()

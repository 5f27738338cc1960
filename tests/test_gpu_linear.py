"""GPU parity of the bare projection (moa_linear) at the row counts and widths of a decoding program against the oracle's
projection: the bf16 matrix kernel in its tiles with and without slices of K, the single-precision kernels, the generic one.
The edges of the bf16 kernel's tiles are in test_gpu_gemm_tiles.py."""
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


# (dtype, rows, K, N)
CASES = [
    ("bf16", 1, 4096, 4096),      # one row
    ("bf16", 33, 4096, 8192),     # just above the 32-row tiles
    ("bf16", 64, 1024, 16384),    # short K, many features
    ("bf16", 60, 2048, 4096),     # the LSA output projection with the folded memory K / V
    ("bf16", 60, 14336, 4096),    # K in slices
    ("bf16", 60, 4096, 10240),    # the grouped projections of a step
    ("bf16", 64, 4096, 28672),    # gate and up projections
    ("bf16", 5, 2048, 14336),     # a few rows
    ("bf16", 47, 4096, 6208),     # a ragged last feature tile
    ("bf16", 65, 4096, 4096),     # a second row tile with one row
    ("bf16", 128, 2048, 2048),
    ("bf16", 160, 2048, 6144),    # three row tiles
    ("bf16", 193, 2048, 2048),    # one row more than K is cut for
    ("bf16", 700, 512, 1024),
    ("bf16", 60, 4096, 1024),     # few features: K in slices
    ("bf16", 17, 384, 96),        # features in 32s
    ("bf16", 9, 200, 50),         # K a multiple of 8 only: single-precision kernels
    ("f32", 19, 320, 70),
]


@pytest.mark.parametrize("dtype,R,K,N", CASES)
def test_linear_parity(G, moa, oracle, dtype, R, K, N):
    rng = np.random.default_rng(R * 7 + K + N)
    x = mi.quantize(rng.standard_normal((R, K)).astype(np.float32), dtype)
    w = mi.quantize((rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32), dtype)
    print(f"[case] linear {dtype} R={R} K={K} N={N}", flush=True)
    mdt = G.MDT[dtype]
    y = torch.full((R, N), float("nan"), dtype=G.TDT[dtype], device="cuda")
    ws = torch.empty(max(moa.linear_workspace_bytes(mdt, R, K, N), 256), dtype=torch.uint8, device="cuda")
    moa.linear(G.dev(x, dtype), G.dev(w, dtype), y, ws)
    torch.cuda.synchronize()
    want = oracle.linear(x, w)
    G.check_close(G.host(y), want, dtype, f"linear[{dtype} {R}x{K}x{N}]", residual_stream=True)
    # the same call again gives the same bits (fixed summation order whatever the scheduling)
    y2 = torch.empty_like(y)
    moa.linear(G.dev(x, dtype), G.dev(w, dtype), y2, ws)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)

"""Helpers for the GPU parity tests: move seeded numpy inputs to the device, run the library through
its binding, bring results back as fp64.  Holds none of the method's arithmetic."""
from __future__ import annotations

import numpy as np
import torch

import moa_inputs as mi
import paper_2410_03804_amd as moa

TDT = {"f32": torch.float32, "bf16": torch.bfloat16}
MDT = {"f32": moa.F32, "bf16": moa.BF16}
# absolute bounds (max-abs against the fp64 oracle): fp32 and bf16 storage
ABS_TOL = {"f32": 1e-4, "bf16": 2e-2}
# tighter relative bound (max-abs / rms of the oracle): a few units of the storage type's rounding step, times the
# growth of rounding error over the sums on the path
REL_TOL = {"f32": 5e-5, "bf16": 3e-2}


def dev(x, dtype=None):
    """numpy -> cuda tensor.  Float arrays hold values already representable in `dtype`."""
    if x is None:
        return None
    t = torch.from_numpy(np.ascontiguousarray(x))
    if dtype is not None:
        t = t.to(TDT[dtype])
    return t.cuda()


def host(t):
    return t.detach().to("cpu", torch.float64).numpy() if t.is_floating_point() else t.cpu().numpy()


def shape_of(cfg: mi.Config):
    return moa.Shape(cfg.L, cfg.d, cfg.H, cfg.Hkv, cfg.dh, cfg.d_lsa_in, cfg.lsa_heads, cfg.Hkv, MDT[cfg.dtype])


def workspace(shape, B, P_cap, M, T):
    n = moa.workspace_bytes(shape, B, P_cap, M, T)
    return torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")


def status_word():
    return torch.zeros(1, dtype=torch.int32, device="cuda")


def launches_of(call):
    """(site, kernel) of each launch that a call makes, as the library's profiler prints them; the call has finished."""
    moa.profile_enable(True)
    try:
        call()
        torch.cuda.synchronize()
        return [(site, kernel) for site, kernel, n, _ in moa.profile_collect() for _ in range(n)]
    finally:
        moa.profile_enable(False)


def kernels_of(call):
    return {kernel for _, kernel in launches_of(call)}


def mask_u64(mask_t):
    return mask_t.cpu().numpy().view(np.uint64)


# A residual stream is not confined to |y| < 2: one bf16 rounding of a value in [4, 8) is already 1.6e-2.  Where a
# result is of that kind (the decoder layer: output rounded once, rotated keys twice), the absolute bound holds up
# to |y| = 2 and becomes this relative one above (bf16: 2^-9 per rounding, a few roundings; fp32 likewise scaled)
BIG_VALUE_REL = {"f32": 5e-5, "bf16": 1e-2}


def check_close(got, want, dtype, what, residual_stream=False, stages=1):
    got = np.asarray(got, dtype=np.float64)
    want = np.asarray(want, dtype=np.float64)
    assert got.shape == want.shape, (what, got.shape, want.shape)
    assert np.all(np.isfinite(got)), f"{what}: non-finite output"
    diff = np.abs(got - want)
    err = float(np.max(diff)) if got.size else 0.0
    rms = float(np.sqrt(np.mean(want ** 2))) if got.size else 1.0
    rel = err / max(rms, 1e-30)
    print(f"[parity] {what}: max-abs {err:.3e}  rms(oracle) {rms:.3e}  max-abs/rms {rel:.3e}", flush=True)
    # stages > 1: the value went through that many residual blocks one after the other, each of which stores its
    # result in the storage type and hands it on, so each adds its own rounding to the stream it inherits
    if residual_stream:
        bound = stages * np.maximum(ABS_TOL[dtype], BIG_VALUE_REL[dtype] * np.abs(want))
        worst = float(np.max(diff / bound)) if got.size else 0.0
        assert worst <= 1.0, f"{what}: error {worst:.2f} x the bound {stages} * max({ABS_TOL[dtype]}, {BIG_VALUE_REL[dtype]} |y|)"
    else:
        assert err <= ABS_TOL[dtype], f"{what}: max-abs {err:.3e} > {ABS_TOL[dtype]}"
    assert rel <= stages * REL_TOL[dtype], f"{what}: max-abs/rms {rel:.3e} > {stages} * {REL_TOL[dtype]}"
    return err, rel


def sample_sequences(plen, n):
    """Indices of n sequences that include the shortest and the longest prefix."""
    order = np.argsort(plen, kind="stable")
    pick = {int(order[0]), int(order[-1])}
    for b in order[len(order) // 2:]:
        if len(pick) >= n:
            break
        pick.add(int(b))
    return sorted(pick)


def slice_step_work(work, seqs):
    """The step workload restricted to the sequences `seqs` (indexing only): every sequence of a step is independent
    of the others, so the oracle's result on the slice is exact for the rows it covers.  Returns the sliced workload
    and the rows of the full LSA input / output that belong to it."""
    cfg = work["cfg"]
    seqs = list(seqs)
    off = work["tok_off"]
    rows = np.concatenate([np.arange(off[b], off[b + 1]) for b in seqs]).astype(np.int64)
    counts = [int(off[b + 1] - off[b]) for b in seqs]
    sub = dict(work)
    sub["cfg"] = mi.scaled(cfg, B=len(seqs))
    for k in ("parent", "tok", "tgt", "prefix_len", "ca_xq", "ca_k", "ca_v", "ca_len0"):
        sub[k] = work[k][seqs]
    sub["lsa_hs"] = work["lsa_hs"][rows]
    sub["tok_off"] = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    sub["layers"] = [dict(w=lay["w"], x=lay["x"][seqs], kcache=lay["kcache"][seqs], vcache=lay["vcache"][seqs])
                     for lay in work["layers"]]
    if work.get("sa") is not None:
        sa = work["sa"]
        sub["sa"] = dict(w=sa["w"], emb=sa["emb"][seqs], kcache=sa["kcache"][seqs], vcache=sa["vcache"][seqs])
    return sub, rows

"""Verification layers of a step in common launches: as many as the workspace has room for, and none whose memory meets another's."""
import numpy as np
import pytest
import torch

import moa_inputs as mi

pytestmark = pytest.mark.gpu

SMALL = dict(B=3, P_min=80, P_max=300, M=37, D=5, max_branch=4, L=6, rms_norm=True)
CFGS = {
    "bf16": mi.Config(name="VG", index=31, dtype="bf16", d=512, H=8, Hkv=2, dh=128, d_lsa_in=512, **SMALL),
    "f32": mi.Config(name="VGf", index=32, dtype="f32", d=256, H=4, Hkv=2, dh=64, d_lsa_in=256, **SMALL),
    # a key range that is split: 15 x 4 x ceil(4 x 37 / 32) = 300 workgroups, more than the whole-range form takes.  148 rows per KV head: one or two
    # calls in a launch take 128-row tiles, five would take 256-row ones.
    "bf16_split": mi.Config(name="VGs", index=33, dtype="bf16", B=15, P_min=120, P_max=220, M=37, D=5, max_branch=4, L=4, d=512, H=16, Hkv=4, dh=128,
                            d_lsa_in=512, rms_norm=True),
}
CFGS["bf16_wide"] = CFGS["bf16_split"]                # the same in 256-row tiles, by the switch for tests
CORES = {"bf16": {"k_attn_fused16<128, 8>", "k_attn_fused<128, 8>"}, "f32": {"k_attn_f32"}, "bf16_split": {"k_attn_mfma<128, 1>", "k_attn_merge<128>"},
         "bf16_wide": {"k_attn_long<128>", "k_attn_merge<128>"}}
SCHEDULES = {"grouped": 0, "two_stream": 1, "sequential": 2}


@pytest.fixture(scope="module")
def G():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_util
    return gpu_util


def apart(step):
    pass


def chained(step):                 # every layer reads what the one before it wrote
    step.v_x = [step.v_x[0]] + step.v_out[:-1]


def one_slab(step):                # all layers' tree keys in the same buffers, the last one's stay
    step.v_ktree = [step.v_ktree[0]] * len(step.v_ktree)
    step.v_vtree = [step.v_vtree[0]] * len(step.v_vtree)


def reads_drafted(step):           # the third layer reads the cross-attention's output
    step.v_x[2] = step.ca_out


def reads_self_attention(step):    # the first layer reads the Self-Attention layer's output
    step.v_x[0] = step.sa["out"]


def unaligned_weight(step):        # the second layer's projection can only be read eight bytes at a time
    w = step.v_w[1]["wk"]
    odd = torch.empty(w.numel() + 4, dtype=w.dtype, device="cuda")[4 if w.element_size() == 2 else 2:][:w.numel()].view(w.shape)
    odd.copy_(w)
    step.v_w[1]["wk"] = odd


def least_workspace(G, step, schedule):
    """The smallest workspace (to 4 KB) in which the step still groups: one verification layer beside the cross-attention."""
    def grouped(n):
        step.ws, step._plans = whole[:n], {}
        G.moa.profile_enable(True)
        try:
            step.run(schedule=schedule)
            torch.cuda.synchronize()
            return any(site == "ca.core+verify.core" for site, *_ in G.moa.profile_collect())
        except G.moa.MoaError:
            return False
        finally:
            G.moa.profile_enable(False)
    whole = step.ws
    lo, hi = 0, whole.numel() // 4096
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if grouped(4096 * mid) else (mid, hi)
    return 4096 * hi


CHANGES = [(f, sa) for f in (apart, chained, one_slab, reads_drafted, reads_self_attention, unaligned_weight) for sa in (False, True) if sa or f is not reads_self_attention]


@pytest.mark.parametrize("change,with_sa", CHANGES, ids=[f.__name__ + "-sa" * sa for f, sa in CHANGES])
@pytest.mark.parametrize("cfg", list(CFGS))
def test_grouped_layers_give_what_one_after_another_gives(G, cfg, change, with_sa):
    """Six layers (a group of four beside the cross-attention at most, then one of two) against the sequential schedule: the same
    bits -- but for the cross-attention and the first layer where the key range is split, whose tiles may be others than those of
    a call alone: to rounding, and the same bits however much room the workspace has."""
    from paper_2410_03804_amd.workload import DeviceStep
    c = CFGS[cfg]
    work = mi.step_workload(c, n_verify_layers=6, with_sa=with_sa)
    outs, cores, sites = {}, {}, {}
    G.moa.debug_force_attn_kernel("split_wide" if cfg == "bf16_wide" else "auto")
    try:
        probe = DeviceStep(work, fold=False)
        need = probe.ws.numel()
        least = least_workspace(G, probe, SCHEDULES["grouped"])
        for name in ("sequential", "grouped", "two_stream", "grouped, as asked for", "two_stream, as asked for", "grouped, least", "two_stream, least"):
            if with_sa and name == "two_stream, least":
                continue                       # (needs more room than grouping does)
            if change in (reads_drafted, reads_self_attention) and with_sa and name.startswith("two_stream"):
                continue                       # there the drafter's layers are another branch than the verification layers
            print(f"[case] verify groups {cfg} {change.__name__} sa={with_sa} {name}", flush=True)
            step = DeviceStep(work, fold=False)
            change(step)
            spare = 5 * 3 * (2 * c.B * c.M * c.H * c.dh * 4 + (1 << 20))
            step.ws = torch.empty(least if "least" in name else need if "asked" in name else need + spare, dtype=torch.uint8, device="cuda")
            launched = G.launches_of(lambda: step.run(schedule=SCHEDULES[name.split(",")[0]]))
            cores[name], sites[name] = [kernel for _, kernel in launched if kernel in CORES[cfg]], {site for site, _ in launched}
            assert step.dev_status.item() == 0
            outs[name] = [t.clone() for t in (step.v_out[0], step.ca_out, *step.v_out[1:], *step.v_ktree, *step.v_vtree, step.mask, step.path, step.bonus)]
    finally:
        G.moa.debug_force_attn_kernel("auto")
    for name, out in outs.items():
        for i, (a, b) in enumerate(zip(outs["sequential"], out)):
            if CORES[cfg] & {"k_attn_merge<128>"} and (i < 2 or change in (chained, reads_drafted)):
                assert torch.allclose(a.float(), b.float(), atol=G.ABS_TOL[c.dtype], rtol=G.REL_TOL[c.dtype]), (name, i)
            else:
                assert torch.equal(a, b), (name, i)
        like = name.split(",")[0] if with_sa else "sequential" if name == "sequential" else "grouped"
        assert all(torch.equal(a, b) for a, b in zip(outs[like], out)), (name, like)
    assert np.isfinite(outs["grouped"][0].float().cpu().numpy()).all()
    # cores launched: one a layer and the drafter's; with room two groups (where the key range is split the first two may have tiles of
    # their own); one by one behind the first two where layers meet, or where there is room for one
    each = 2 if "k_attn_merge<128>" in CORES[cfg] else 1
    n = {name: len(got) for name, got in cores.items()}
    assert n["sequential"] == (7 + with_sa) * each, cores
    assert n["grouped, least"] == (6 + with_sa) * each, cores
    if change is apart:
        assert (2 + with_sa) * each <= n["grouped"] <= (2 + with_sa + each - 1) * each, cores
    if change in (chained, one_slab):
        assert n["grouped"] == (6 + with_sa) * each, cores
    # the Self-Attention layer's projections: in the first launch, unless a layer in it reads what that layer writes
    if with_sa and change is reads_self_attention:
        assert "sa.qkv_proj" in sites["grouped"], sites
    if with_sa and change is apart and cfg == "f32":
        assert "sa.qkv_proj" not in sites["grouped"], sites


# Shapes where the Self-Attention layer's projections in a launch with the verification layers' would take another kernel than alone,
# or take the verification layers' to one: (step, query heads and KV heads of the layer)
SELF = {
    # fp32, 64 + 4 + 4 tiles of 64 features alone, twice the 64 in a launch of the step: on either side of 128
    "f32_wide": (mi.Config(name="VSw", index=34, dtype="f32", B=1, P_min=30, P_max=60, M=20, D=4, max_branch=4, L=4, d=256, H=64, Hkv=4, dh=64,
                           d_lsa_in=256, rms_norm=True), 64, 4),
    # fp32, a layer four times as wide as the others
    "f32_wider": (mi.Config(name="VSv", index=35, dtype="f32", B=1, P_min=30, P_max=60, M=20, D=4, max_branch=4, L=4, d=256, H=16, Hkv=4, dh=64,
                            d_lsa_in=256, rms_norm=True), 64, 8),
    # bf16, 16 key features, which the bf16 matrix kernels do not take
    "bf16_narrow": (mi.Config(name="VSn", index=36, dtype="bf16", B=2, P_min=30, P_max=60, M=20, D=4, max_branch=4, L=4, d=256, H=8, Hkv=2, dh=16,
                              d_lsa_in=256, rms_norm=True), 8, 1),
    # bf16, long K and few features: slices of K alone
    "bf16_sliced": (mi.Config(name="VSs", index=37, dtype="bf16", B=1, P_min=30, P_max=60, M=8, D=4, max_branch=4, L=4, d=8192, H=2, Hkv=1, dh=128,
                              d_lsa_in=256, rms_norm=True), 2, 1),
    # no such edge: shares the launch
    "bf16": (mi.Config(name="VSb", index=38, dtype="bf16", B=1, P_min=30, P_max=60, M=12, D=4, max_branch=4, L=4, d=4096, H=32, Hkv=8, dh=128,
                       d_lsa_in=1024, rms_norm=True), 32, 8),
}


@pytest.mark.parametrize("case", list(SELF))
def test_self_attention_in_a_step_gives_what_the_call_alone_gives(G, case):
    """Under every schedule, and the verification layers what they give without it."""
    from paper_2410_03804_amd.workload import DeviceStep
    moa = G.moa
    c, H, hkv = SELF[case]
    work = mi.step_workload(c, n_verify_layers=2, with_sa=True)
    dt, rng = c.dtype, np.random.default_rng(c.index)
    zeros = lambda *shape: torch.zeros(shape, dtype=G.TDT[dt], device="cuda")
    w = {k: rng.standard_normal(s) * s[1] ** -0.5 for k, s in (("wq", (H * c.dh, c.d)), ("wk", (hkv * c.dh, c.d)), ("wv", (hkv * c.dh, c.d)), ("wo", (c.d, H * c.dh)))}
    sa = dict(shape=moa.Shape(c.L, c.d, H, hkv, c.dh, c.d_lsa_in, c.lsa_heads, c.Hkv, G.MDT[dt]), emb=G.dev(work["sa"]["emb"], dt), w={k: G.dev(v, dt) for k, v in w.items()},
              kcache=zeros(c.B, hkv, c.P_cap, c.dh).normal_(), vcache=zeros(c.B, hkv, c.P_cap, c.dh).normal_(), P_cap=c.P_cap)
    outs, sites = {}, {}
    for name, schedule in SCHEDULES.items():
        print(f"[case] self-attention in a step {case} {name}", flush=True)
        step = DeviceStep(work, fold=False)
        step.sa = dict(sa, k_draft=zeros(c.B, hkv, c.M, c.dh), v_draft=zeros(c.B, hkv, c.M, c.dh), out=zeros(c.B, c.M, c.d))
        step.ws = torch.empty(2 * max(step.ws.numel(), moa.workspace_bytes(sa["shape"], c.B, c.P_cap, c.M, 0)), dtype=torch.uint8, device="cuda")
        moa.profile_enable(True)
        step.run(schedule=schedule)
        torch.cuda.synchronize()
        sites[name] = {site for site, *_ in moa.profile_collect()}
        moa.profile_enable(False)
        assert step.dev_status.item() == 0
        outs[name] = [t.clone() for t in (step.sa["out"], step.sa["k_draft"], step.sa["v_draft"], *step.v_out, *step.v_ktree, *step.v_vtree)]
    alone = [torch.zeros_like(t) for t in outs["grouped"][:3]]
    moa.self_attn_draft(sa["shape"], sa["emb"], 0, *(sa["w"][k] for k in ("wq", "wk", "wv", "wo")), sa["kcache"], sa["vcache"], step.prefix_len, c.P_cap, step.mask,
                        *alone, G.workspace(sa["shape"], c.B, c.P_cap, c.M, 0), G.status_word())
    torch.cuda.synchronize()
    for name, out in outs.items():
        for i, (a, b) in enumerate(zip(alone + outs["sequential"][3:], out)):
            assert torch.equal(a, b), (name, i)
    assert ("sa.qkv_proj" in sites["grouped"]) == (case != "bf16"), sites


def test_the_smaller_capacity_may_need_more_scratch(G):
    """The cross-attention over the whole of 8192 keys, two verification layers in slices of 8065, which take more scratch than slices of
    8192 would: no core falls back to the kernel that needs none, and the results are those of one stage after another."""
    from paper_2410_03804_amd.workload import DeviceStep
    c = mi.Config(name="VSc", index=39, dtype="bf16", B=4, P_min=7000, P_max=7937, M=128, D=6, max_branch=4, L=4, d=512, H=11, Hkv=1, dh=128, d_lsa_in=256,
                  rms_norm=True)
    work = mi.step_workload(c, n_verify_layers=2)
    assert work["P_cap"] == 8065
    for k in ("ca_k", "ca_v"):
        old = work[k]
        work[k] = np.zeros((c.B, c.Hkv, 8192, c.dh), dtype=old.dtype)
        work[k][:, :, :old.shape[2]] = old
    work["ca_P_cap"] = 8192
    outs = {}
    for name, schedule in SCHEDULES.items():
        print(f"[case] capacities 8192 and 8065 {name}", flush=True)
        step = DeviceStep(work, fold=False)
        launched = G.launches_of(lambda: step.run(schedule=schedule))
        kernels = {kernel for site, kernel in launched if "core" in site}
        assert "k_attn_generic" not in kernels and any(k.startswith("k_attn_fused") for k in kernels) and "k_attn_merge<128>" in kernels, (name, kernels)
        assert step.dev_status.item() == 0
        outs[name] = [t.clone() for t in (*step.v_out, step.ca_out)]
    for out in outs.values():
        assert all(torch.equal(a, b) for a, b in zip(outs["sequential"], out))

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
    # a key range that is split (16 sequences, too many workgroups for the whole-range form)
    "bf16_split": mi.Config(name="VGs", index=33, dtype="bf16", B=16, P_min=300, P_max=700, M=60, D=6, max_branch=4, L=4, d=512, H=8, Hkv=4, dh=128,
                            d_lsa_in=512, rms_norm=True),
}
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
    if step.sa:
        step.v_x[0] = step.sa["out"]


def unaligned_weight(step):        # the second layer's projection can only be read eight bytes at a time
    w = step.v_w[1]["wk"]
    odd = torch.empty(w.numel() + 4, dtype=w.dtype, device="cuda")[4 if w.element_size() == 2 else 2:][:w.numel()].view(w.shape)
    odd.copy_(w)
    step.v_w[1]["wk"] = odd


@pytest.mark.parametrize("with_sa", [False, True], ids=["", "sa"])
@pytest.mark.parametrize("change", [apart, chained, one_slab, reads_drafted, reads_self_attention, unaligned_weight], ids=lambda f: f.__name__)
@pytest.mark.parametrize("cfg", list(CFGS))
def test_grouped_layers_give_what_one_after_another_gives(G, cfg, change, with_sa):
    """Six layers (a group of four beside the cross-attention at most, then one of two) against the sequential schedule: the same
    bits where the attention runs over the whole key range in one form, to rounding where the key range is split."""
    from paper_2410_03804_amd.workload import DeviceStep
    c = CFGS[cfg]
    work = mi.step_workload(c, n_verify_layers=6, with_sa=with_sa)
    need = None
    outs = {}
    for name in ("sequential", "grouped", "two_stream", "grouped, no room to spare", "two_stream, no room to spare"):
        if change in (reads_drafted, reads_self_attention) and with_sa and name.startswith("two_stream"):
            continue                       # there the drafter's layers are another branch than the verification layers
        print(f"[case] verify groups {cfg} {change.__name__} sa={with_sa} {name}", flush=True)
        step = DeviceStep(work, fold=False)
        change(step)
        need = need or step.ws.numel()
        spare = 0 if "no room" in name else 5 * 3 * (2 * c.B * c.M * c.H * c.dh * 4 + (1 << 20))
        step.ws = torch.empty(need + spare, dtype=torch.uint8, device="cuda")
        step.run(schedule=SCHEDULES[name.split(",")[0]])
        torch.cuda.synchronize()
        assert step.dev_status.item() == 0
        outs[name] = [t.clone() for t in (*step.v_out, *step.v_ktree, *step.v_vtree, step.ca_out, step.mask, step.path, step.bonus)]
    for name, out in outs.items():
        for i, (a, b) in enumerate(zip(outs["sequential"], out)):
            if cfg == "bf16_split":
                assert torch.allclose(a.float(), b.float(), atol=G.ABS_TOL[c.dtype], rtol=G.REL_TOL[c.dtype]), (name, i)
            else:
                assert torch.equal(a, b), (name, i)
    assert np.isfinite(outs["grouped"][0].float().cpu().numpy()).all()

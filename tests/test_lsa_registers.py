"""Scratch memory in the assembly the compiler makes of the one-kernel Layer Self-Attention (gfx950 only, no GPU needed): these
kernels fill the register file, and a value that no longer fits shows up as scratch traffic, not as an error."""
import re
import subprocess

import pytest

from paper_2410_03804_amd import build


@pytest.fixture(scope="module")
def kernels():
    cmd = [build._hipcc(), *build.FLAGS, "--cuda-device-only", "-S", "-o", "-", str(build.CSRC / "moa_lsa_fused.hip")]
    asm = subprocess.run(cmd, capture_output=True, text=True, check=True).stdout
    found = re.findall(r"^(_ZN3moa\d+k_lsa_fused\w*):(.*?)\.end_amdhsa_kernel", asm, re.M | re.S)
    assert len(found) >= 16
    return dict(found)


def test_only_the_dense_form_spills_registers(kernels):
    size = {name: int(re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", body).group(1)) for name, body in kernels.items()}
    assert not {name: n for name, n in size.items() if n and "_pk_dense" not in name}


def test_no_spill_inside_the_k_loop(kernels):
    """160 rows of accumulators leave no register over: what the dense form spills, it stores before the loop over the input
    width and loads behind it."""
    for name, body in kernels.items():
        loops, label_at = [], {}
        for m in re.finditer(r"^(\.LBB\w+):|^\ts_c?branch\w* (\.LBB\w+)$", body, re.M):
            if m.group(1):
                label_at[m.group(1)] = m.end()
            elif m.group(2) in label_at:                   # a branch back: from its target to here is a loop
                loops.append(body[label_at[m.group(2)]:m.start()])
        loops = [text for text in loops if "v_mfma" in text and "s_barrier" in text]
        assert loops and not any("scratch_" in text for text in loops), name

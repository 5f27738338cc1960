"""The direct global -> LDS loads that are written as inline asm, in the assembly the compiler makes of the kernels that use
them (gfx950 only, no GPU needed)."""
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2410_03804_amd import build

SOURCES = ["moa_gemm_bf16.hip", "moa_lm_head.hip", "moa_attn_long.hip"]


@pytest.fixture(scope="module")
def asm():
    def compile_one(src):
        cmd = [build._hipcc(), *build.FLAGS, *build.SOURCE_FLAGS.get(src, []), "--cuda-device-only", "-S", "-o", "-", str(build.CSRC / src)]
        return subprocess.run(cmd, capture_output=True, text=True, check=True).stdout
    with ThreadPoolExecutor(3) as ex:
        return dict(zip(SOURCES, ex.map(compile_one, SOURCES)))


@pytest.mark.parametrize("src", SOURCES)
def test_base_address_of_lds_loads_comes_from_a_scalar_move(asm, src):
    """A vector memory instruction must not read a scalar that a vector instruction wrote less than five wait states before
    (a register restored from a spill lane); a scalar move in between waits for it.  It also stands between the write of m0
    and its use.  m0 holds nothing else in these kernels."""
    lines = [l.split(";")[0].strip() for l in asm[src].splitlines()]
    lines = [l for l in lines if l and not l.startswith(".")]
    loads = [i for i, l in enumerate(lines) if l.startswith("global_load_lds_dwordx4")]
    assert loads
    for i in loads:
        base = re.fullmatch(r"global_load_lds_dwordx4 v\d+, (s\[\d+:\d+\])", lines[i]).group(1)
        assert re.fullmatch(rf"s_mov_b64 {re.escape(base)}, (s\[\d+:\d+\]|vcc)", lines[i - 1]), lines[i - 2:i + 1]
        assert re.fullmatch(r"s_mov_b32 m0, (s\d+|vcc_lo|vcc_hi|\w+)", lines[i - 2]), lines[i - 2:i + 1]
    assert sum(bool(re.search(r"\bm0\b", l)) for l in lines) == len(loads)

"""The binding's check of one tensor argument (csrc/argcheck.c).  A tensor that says it is on the GPU stands in for one."""
import shutil
import subprocess
import sys
from pathlib import Path

import pytest
import torch

import paper_2410_03804_amd as moa
from paper_2410_03804_amd.binding import _dev


class OnGpu(torch.Tensor):
    is_cuda = True


def gpu(*shape, dtype=torch.int32):
    return torch.zeros(*shape, dtype=dtype).as_subclass(OnGpu)


def test_address_of_what_a_call_can_use():
    t = gpu(4, 6)
    assert _dev(t, torch.int32, 24, "x") == t.data_ptr() and _dev(t, torch.int32, 0, "x") == t.data_ptr()
    assert _dev(None, torch.int32, 24, "x") is None


@pytest.mark.parametrize("arg,dtype,numel,error,text", [
    (3, torch.int32, 1, TypeError, "x: expected a torch tensor"),
    (torch.zeros(4, dtype=torch.int32), torch.int32, 1, ValueError, "x: must be a contiguous CUDA tensor"),
    (gpu(4, 6).t(), torch.int32, 24, ValueError, "x: must be a contiguous CUDA tensor"),
    (gpu(4, dtype=torch.float32), torch.int32, 4, ValueError, "x: dtype torch.float32, expected torch.int32"),
    (gpu(4, 6), torch.int32, 25, ValueError, "x: 24 elements, the call touches 25"),
    (gpu(4, 6), torch.int32, 1 << 70, ValueError, "x: 24 elements, the call touches 1180591620717411303424")])
def test_what_it_refuses(arg, dtype, numel, error, text):
    with pytest.raises(error) as e:
        _dev(arg, dtype, numel, "x")
    assert str(e.value) == text


def test_errors_of_its_arguments_pass_through():
    with pytest.raises(TypeError):
        _dev(gpu(4), torch.int32, "four", "x")
    with pytest.raises(TypeError):
        _dev(gpu(4), torch.int32, 4)


@pytest.mark.parametrize("missing", ["libmoa.so", "_argcheck.abi3.so"])
def test_what_is_not_built_says_how_to_build_it(tmp_path, missing):
    """In a copy of the package that lacks one of the two built files, or has one that is no extension."""
    here, pkg = Path(moa.library_path()).parent, tmp_path / "paper_2410_03804_amd"
    pkg.mkdir()
    for f in (*here.glob("*.py"), *here.glob("*.so")):
        if f.name != missing:
            shutil.copy(f, pkg)
    for broken in (False, True):
        if broken:
            (pkg / "_argcheck.abi3.so").write_bytes(b"not an extension")
        r = subprocess.run([sys.executable, "-c", "import paper_2410_03804_amd"], cwd=tmp_path, capture_output=True, text=True)
        assert r.returncode != 0 and "build.py` (there is no fallback path)" in r.stderr and f"ImportError: {pkg}" in r.stderr, r.stderr

"""The binding's check of one tensor argument (csrc/argcheck.c).  A tensor that says it is on the GPU stands in for one."""
import pytest
import torch

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

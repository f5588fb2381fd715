"""Adam's square root: the build asks for correctly rounded roots (CPU), and
on the GPU the compiler's root and the checked one are the correctly rounded
root for all 2^32 fp32 values."""

import ctypes

import pytest

from paper_1805_07891_amd import build


def test_the_build_asks_for_correctly_rounded_roots():
    assert "-fhip-fp32-correctly-rounded-divide-sqrt" in build.FLAGS


@pytest.mark.gpu
def test_both_roots_are_correctly_rounded_for_every_value():
    import torch
    lib = ctypes.CDLL(build.ROOTS_LIB)
    lib.phub_check_roots.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    wrong = torch.zeros(2, dtype=torch.int64, device="cuda:0")
    torch.cuda.synchronize()
    print("roots of 2^32 values", flush=True)
    assert lib.phub_check_roots(None, None) == -1
    assert lib.phub_check_roots(wrong.data_ptr(), None) == 0
    torch.cuda.synchronize()
    assert wrong.tolist() == [0, 0]

"""CPU: the native part of the binding hands the library what ctypes would, and leaves every unusual call to it."""
import ctypes as C

import pytest

import paper_2508_06041_amd as dp
from paper_2508_06041_amd import binding

calls = binding._calls


class Tensor:
    """As much of a tensor as the binding looks at."""

    def __init__(self, address, *shape):
        self.address, self.shape = address, shape

    def data_ptr(self):
        return self.address

    def dim(self):
        return len(self.shape)

    def size(self, i):
        return self.shape[i]


@pytest.fixture
def made():
    """Every call of the library functions, which stand-ins take here."""
    got = []
    vp, i32 = C.c_void_p, C.c_int
    gemv = C.CFUNCTYPE(i32, vp, i32, i32, vp, vp, vp, i32, vp)(lambda *a: got.append(a) or -3)
    estimate = C.CFUNCTYPE(i32, vp, i32, i32, i32, vp, vp, vp, vp)(lambda *a: got.append(a) or -2)
    calls.bind(C.cast(gemv, vp).value, C.cast(estimate, vp).value, lambda: 5, lambda device: 1000 + device)
    yield got
    import torch
    calls.bind(C.cast(binding.lib.dpllm_gemv, vp).value, C.cast(binding.lib.dpllm_estimate, vp).value,
               torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)


def test_arguments_arrive(made):
    x, y, kd, high = Tensor(64, 32), Tensor(128, 8), Tensor(256, 1), Tensor(2 ** 63 + 64, 3, 32)
    assert calls.gemv(7, 2, 4, x, y, None) == -3
    assert calls.gemv(2 ** 47, -1, -1, high, y, kd) == -3
    assert calls.gemv(7, 2 ** 32 + 5, True, Tensor(0, 8, 32), y, None) == -3      # as ctypes converts an int
    assert made == [(7, 2, 4, None, 64, 128, 1, 1005), (2 ** 47, -1, -1, 256, 2 ** 63 + 64, 128, 3, 1005), (7, 5, 1, None, None, 128, 8, 1005)]
    made.clear()
    assert calls.estimate(7, 1, 3, 4, x, y, kd) == -2
    assert made == [(7, 1, 3, 4, 64, 128, 256, 1005)]


@pytest.mark.parametrize("change", [{0: 0}, {0: None}, {1: 1.0}, {2: "3"}, {3: 64}, {3: None}, {3: Tensor(64)}, {4: None}, {4: 128}, {5: 256}, {5: object()}])
def test_unusual_calls_are_made_elsewhere(made, change):
    args = [7, 2, 4, Tensor(64, 32), Tensor(128, 8), Tensor(256, 1)]
    for i, v in change.items():
        args[i] = v
    assert calls.gemv(*args) == calls.ELSEWHERE
    if 3 not in change or change[3] is None:        # (the sample count is no business of an estimate)
        assert calls.estimate(args[0], args[1], args[2], 4, args[3], args[4], args[5] if 5 in change else Tensor(256, 1)) == calls.ELSEWHERE
    assert made == []


def test_errors_of_a_failing_lookup_do_not_stay(made):
    class Broken(Tensor):
        def data_ptr(self):
            raise RuntimeError("no storage")
    assert calls.gemv(7, 2, 4, Broken(64, 32), Tensor(128, 8), None) == calls.ELSEWHERE
    assert made == []
    assert dp.DPLLM_OK == 0

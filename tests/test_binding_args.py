"""What the Python binding hands to the C boundary for each form of argument it takes (no GPU)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2605_06472_amd import binding


def _read(address, n):
    if not isinstance(address, int):                  # byref(): ctypes converts it as it converts an address
        address = ctypes.cast(address, ctypes.c_void_p).value
    return list((ctypes.c_int32 * n).from_address(address)) if n else []


def _read_only():
    a = np.arange(5, dtype=np.int32)
    a.setflags(write=False)
    return a


@pytest.mark.parametrize("form", [
    lambda: np.arange(5, dtype=np.int32), _read_only, lambda: np.arange(10, dtype=np.int32)[::2] // 2,
    lambda: (np.arange(15, dtype=np.int32) // 3)[::3], lambda: np.arange(5, dtype=np.int64), lambda: np.arange(5, dtype=">i4"),
    lambda: np.arange(5, dtype=np.int32).reshape(5, 1), lambda: [0, 1, 2, 3, 4], lambda: torch.arange(5, dtype=torch.int32),
    lambda: torch.arange(5, dtype=torch.int64)],
    ids=["plain", "read_only", "computed", "strided", "int64", "big_endian", "2d", "list", "torch", "torch_int64"])
def test_host_lengths_arrive_as_int32(form):
    array, address = binding._host_i32(form())
    assert array.size == 5 and _read(address, 5) == [0, 1, 2, 3, 4]


def test_empty_and_address_arguments():
    array, _ = binding._host_i32(np.zeros(0, np.int32))
    assert array.shape == (0,)
    assert binding._ptr(None) is None and binding._ptr(12345) == 12345
    t = torch.zeros(4)
    assert binding._ptr(t) == t.data_ptr()
    assert binding._stream(77) == 77

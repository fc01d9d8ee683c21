"""Uploading a tree's tables launches a kernel; an error that an earlier call of the program left behind is not that kernel's."""
import ctypes
import re

import numpy as np
import pytest
import torch

import paper_2007_12792_amd as octfd

pytestmark = pytest.mark.gpu


def runtime():
    with open("/proc/self/maps") as f:
        return ctypes.CDLL(re.search(r"\S*/libamdhip64\.so\S*", f.read()).group(0))


def test_upload_after_a_failed_allocation_elsewhere(dev):
    t = octfd.Tree.build(3, 4, np.array([[1000, 2000, 1040000]], np.uint32), np.array([60000], np.uint32))
    torch.zeros(1, device=dev)
    octfd.lib()
    hip = runtime()
    ptr = ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(ptr), ctypes.c_size_t(1 << 60)) == 2 and not ptr.value      # hipErrorOutOfMemory
    try:
        t.upload()
    finally:
        hip.hipGetLastError()                        # the error is this test's: nobody else is to find it
    u = torch.ones((1, t.n, 8, 8, 8), dtype=torch.float64, device=dev)
    padded = torch.zeros((1, t.n, 14, 14, 14), dtype=torch.float64, device=dev)
    t.unzip(u, padded)
    assert ((padded - 1).abs() < 1e-14).all()

"""Registers of the search kernels: the search with Deps of several words
never takes the one-wave rounds, so its state must not be spilled around
their call (compiled with it, a 2000-vertex colouring took 14% longer at
W = 2)."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu


class _Attr(ctypes.Structure):            # hipFuncAttributes
    _fields_ = [("binaryVersion", ctypes.c_int), ("cacheModeCA", ctypes.c_int),
                ("constSizeBytes", ctypes.c_size_t), ("localSizeBytes", ctypes.c_size_t),
                ("maxDynamicSharedSizeBytes", ctypes.c_int), ("maxThreadsPerBlock", ctypes.c_int),
                ("numRegs", ctypes.c_int), ("preferredShmemCarveout", ctypes.c_int),
                ("ptxVersion", ctypes.c_int), ("sharedSizeBytes", ctypes.c_size_t)]


@pytest.mark.parametrize("threads", [64, 128, 256, 512])
@pytest.mark.parametrize("learning", [0, 1])
@pytest.mark.parametrize("extended", [0, 1])
def test_wide_search_keeps_its_state_in_registers(threads, learning, extended):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1909_01786_amd as P
    so = P.lib()
    name = f"_ZN3asp8k_searchILi{threads}ELi{learning}ELi{extended}ELb0EEEvNS_5KArgsE"
    handle = ctypes.c_void_p.in_dll(so, name)
    a = _Attr()
    assert so.hipFuncGetAttributes(ctypes.byref(a), ctypes.byref(handle)) == 0
    assert a.numRegs > 64                     # the attributes are filled in
    assert a.localSizeBytes == 0

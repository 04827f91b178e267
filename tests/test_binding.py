"""Argument marshalling of the ctypes binding, without a GPU: what is no address is refused before the library sees it."""
import ctypes

import numpy as np
import pytest

from paper_2311_03285_amd import slora


@pytest.mark.parametrize("call", ["lora_apply_multi", "lora_apply_multi_y16", "lora_apply_multi_static"])
@pytest.mark.parametrize("bad", [None, ctypes.c_void_p(4096), ctypes.c_uint64(4096), "y", b"y"])
@pytest.mark.parametrize("n", [1, 9])
def test_what_is_no_address_is_refused(call, bad, n):
    good = [4096 * (i + 1) for i in range(n)]
    for xs, ys in ((good[1:] + [bad], good), (good, [bad] + good[1:])):
        with pytest.raises((TypeError, ValueError)):
            getattr(slora, call)(None, np.arange(n, dtype=np.int32), xs, ys)


@pytest.mark.parametrize("slots", [[0, 1, 2], (0, 1, 2), np.arange(3, dtype=np.int32), np.arange(3), np.arange(6, dtype=np.int32)[::2] // 2])
def test_slots_and_addresses_reach_the_library(slots):
    n, got = slora._slot_array(slots)
    assert n == 3 and list(ctypes.cast(got, ctypes.POINTER(ctypes.c_int32))[:3]) == [0, 1, 2]
    for ptrs in ([1 << 47, np.int64(16), True], [np.uint64(1 << 47), 16.0, 1]):
        assert list(ctypes.cast(slora._ptr_array(ptrs), ctypes.POINTER(ctypes.c_uint64))[:3]) == [1 << 47, 16, 1]
    with pytest.raises(slora.SloraError, match="plan is NULL"):
        slora.lora_apply_multi(None, slots, [4096] * 3, [8192] * 3)

"""The binding's raw calls (no GPU needed): a host object in the place of a device
pointer is refused before the library sees it."""
import ctypes

import pytest

from paper_2605_15547_amd import crmath

HOST = [b"\0" * 64, "0" * 64, (ctypes.c_float * 16)(), 1.5]


@pytest.mark.parametrize("host", HOST, ids=lambda h: type(h).__name__)
def test_host_objects_are_no_device_pointers(host):
    for a, b in ((host, 0x2000), (0x1000, host)):
        with pytest.raises(TypeError):
            crmath.eval_ptr("expf", a, b, 8)
    for a, b, c in ((host, 0x2000, 0x3000), (0x1000, host, 0x3000), (0x1000, 0x2000, host)):
        with pytest.raises(TypeError):
            crmath.dft_ptr(a, 8, b, 4, c)

"""The strided passes have instances that carry compiled plans only and do nothing for any other plan, so the host may choose
them only for a plan that they carry and whose tile holds it. The choice is a host function of the library, called here for
every mesh side, width of columns and points per thread that there is an instance of."""
import ctypes

import pytest

STAGES = 7


class Plan1D(ctypes.Structure):
    _fields_ = [("n", ctypes.c_int), ("nst", ctypes.c_int)] + [(f, ctypes.c_int * STAGES)
                                                              for f in ("radix", "p", "pmask", "tw_off")]


def functions():
    from paper_1506_03737_amd import lpc
    make = getattr(lpc.LIB, "_ZN3lpc4kern9make_planEiPNS0_6Plan1DEb")
    make.restype, make.argtypes = ctypes.c_bool, [ctypes.c_int, ctypes.POINTER(Plan1D), ctypes.c_bool]
    fixed = getattr(lpc.LIB, "_ZN3lpc4kern14has_fixed_planERKNS0_6Plan1DEii")
    fixed.restype, fixed.argtypes = ctypes.c_bool, [ctypes.POINTER(Plan1D), ctypes.c_int, ctypes.c_int]
    return make, fixed


@pytest.mark.parametrize("columns", [8, 16, 32])
@pytest.mark.parametrize("points", [8, 12, 16])
def test_compiled_plans_fit(columns, points):
    make, fixed = functions()
    chosen = []
    for n in range(8, 1025, 2):
        p = Plan1D()
        if make(n, ctypes.byref(p), True) and fixed(ctypes.byref(p), columns, points):
            chosen.append(n)
    # the compiled plans' lengths whose points (n columns over 512 threads) the threads hold
    assert chosen == [n for n in (192, 256, 320, 384, 768, 1024) if n * columns <= 512 * points]

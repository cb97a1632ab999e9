import ctypes
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def oracle():
    import oracle as orc

    orc.build()
    return orc


@pytest.fixture(scope="session")
def dispatch_rule():
    """mmoe::name(const mmoe_shape&[, int, bool]), bool or as restype says: a rule of the library's dispatch, by its C++ symbol."""
    from paper_2505_06481_amd import mmoe

    def rule(name, shape, *args, restype=ctypes.c_bool):
        f = getattr(mmoe.lib(), f"_ZN4mmoe{len(name)}{name}ERK10mmoe_shape" + "ib"[:len(args)])
        f.restype = restype
        f.argtypes = [ctypes.c_void_p] + [ctypes.c_int, ctypes.c_bool][:len(args)]
        return f(ctypes.addressof(shape), *args)

    return rule

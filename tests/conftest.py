import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU")
    config.addinivalue_line("markers", "slow: long-running CPU check")


@pytest.fixture(autouse=True)
def untuned():
    """Tuned tile widths are process-wide: every test begins without any, so
    that what one loads or tunes does not choose the kernels of the next."""
    native = sys.modules.get("paper_2012_00506_amd._native")
    if native is not None and native._lib is not None:
        import ctypes as C
        f = native._lib._ZN2fb17set_tuned_variantEmii
        f.restype, f.argtypes = None, [C.c_size_t, C.c_int, C.c_int]
        for rsize in (4, 8):
            for nb in range(16, 129, 16):
                f(rsize, nb, -1)
    yield

import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU; runs the HIP library")
    config.addinivalue_line("markers", "slow: longer CPU-only oracle checks")


@pytest.fixture(scope="session")
def oracle_mod():
    import oracle

    oracle._lib()  # builds fd_oracle.c with gcc if no build is present
    return oracle


@pytest.fixture(autouse=True)
def library_tiles():
    """Tiles set by hand are process-wide: none outlives its test, also one that fails."""
    yield
    F = sys.modules.get("paper_1410_1387_amd.fdwave")
    if F is None or F._lib is None:
        return
    for dtype in ("f32", "f64"):
        for r in range(1, 9):
            for ndim in (2, 3):
                F.fd_set_tuning(dtype, r, ndim, -1)
                F.fd_set_adj_tuning(dtype, r, ndim, -1)
        for rxy in (2, 4, 8, 12):
            for rz in (1, 2, 4, 8):
                if rz <= rxy:
                    F.fd_vti_set_tuning(dtype, rxy, rz, 0, 0)

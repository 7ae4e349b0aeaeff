import os
import sys
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="module", autouse=True)
def memory_given_back():
    """What a module leaves in torch's cache (190 GB after the full-size ones) goes back to the driver before the next one starts.  The
    driver clears it for some seconds, in which a hipFree takes 7 ms for 0.25, in whatever test is being timed then."""
    yield
    torch = sys.modules.get("torch")
    if torch is None or not torch.cuda.is_initialized() or torch.cuda.memory_reserved() < 8 << 30:
        return
    torch.cuda.empty_cache()
    quick, end = 0, time.perf_counter() + 10.0
    while quick < 5 and time.perf_counter() < end:
        block = torch.empty(160 << 20, dtype=torch.uint8, device="cuda")
        del block
        t0 = time.perf_counter()
        torch.cuda.empty_cache()
        quick = quick + 1 if time.perf_counter() - t0 < 2e-3 else 0
        time.sleep(0.05)

"""The 8-byte form of the edge chunks' estimates (grem_es_estimate.hip.h) on the host against Alg. 1's blend in doubles: the same
values bit for bit after every chunk, and the same side ahead."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2502_17846_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("estimates") / "libestimates.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-shared", "-fPIC", "-O2", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I", CSRC, "-o", out,
                    os.path.join(HERE, "edge_estimates.cpp")], check=True)
    return ctypes.CDLL(out)


def _check(lib, h):
    """h: (nodes, chunks, 2) fresh counts.  Returns which nodes' estimates were in doubles, chunk by chunk."""
    h = np.ascontiguousarray(h, np.uint32)
    count, steps, _ = h.shape
    sums, lean, wide = np.full(h.shape, np.nan), np.full((count, steps), 9, np.int32), np.zeros((count, steps), np.uint8)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    lib.run_blends(ctypes.c_int64(count), ctypes.c_int64(steps), p(h), p(sums), p(lean), p(wide))
    est = h[:, 0].astype(np.float64)
    for i in range(steps):
        if i:
            est = (est + h[:, i].astype(np.float64)) * 0.5
        assert np.array_equal(sums[:, i].view(np.uint64), est.view(np.uint64)), i
        assert np.array_equal(lean[:, i], (est[:, 1] > est[:, 0]).astype(np.int32) - (est[:, 0] > est[:, 1])), i
    return wide


def test_ordinary_counts(lib):
    rng = np.random.default_rng(1)
    for most in (2, 40, 3000, 1 << 20, (1 << 32) - 1):
        wide = _check(lib, rng.integers(0, most, (400, 70, 2)))
        assert wide[:, -1].all() and not (most < 40 and wide[:, 20].any())


# halved 28 or 29 times, then so many ends of either side that their sums need more than 53 bits: equal as doubles, though not as whole numbers
@pytest.mark.parametrize("quiet", range(24, 32))
@pytest.mark.parametrize("bits", [22, 23, 24, 25, 28, 31])
def test_sums_that_doubles_round(lib, quiet, bits):
    first = np.array([[a, b] for a in (0, 1, 3) for b in (0, 1, 2, 7)])
    last = np.array([[(1 << bits) + a, (1 << bits) + b] for a in (0, 1, 5) for b in (0, 1, 6)])
    h = np.zeros((len(first) * len(last), quiet + 3, 2), np.uint32)
    h[:, 0] = np.repeat(first, len(last), 0)
    h[:, quiet] = np.tile(last, (len(first), 1))
    h[:, quiet + 1] = 1
    _check(lib, h)

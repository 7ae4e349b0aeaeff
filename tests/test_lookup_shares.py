"""Look-up launches of the two-phase route over column blocks of unequal sizes: every group of tuples is dealt to one workgroup, and no
workgroup's share is much longer than the others'."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2502_17846_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("shares") / "libshares.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-shared", "-fPIC", "-O2", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I", CSRC, "-o", out,
                    os.path.join(HERE, "lookup_shares.cpp")], check=True)
    lib = ctypes.CDLL(out)
    lib.longest_sweep_share.restype = ctypes.c_int64
    return lib


def _sizes():
    rng = np.random.default_rng(2)
    yield "equal", np.full(212, 235_000)
    yield "by degree", (50_000_000 / np.arange(1, 213) ** 0.9 / 12).astype(np.int64)
    yield "one block", np.array([47_000_000])
    yield "all in the last", np.r_[np.zeros(99, np.int64), 10_000_000]
    yield "empty between", np.where(rng.random(4096) < 0.5, 0, rng.integers(0, 30_000, 4096))
    yield "no entries", np.zeros(7, np.int64)
    yield "few", np.array([1, 0, 3, 1023, 1024, 1025])


@pytest.mark.parametrize("name,size", list(_sizes()))
def test_a_sweep_deals_every_group_once_in_even_shares(lib, name, size):
    start = np.zeros(len(size) + 1, np.uint32)
    start[1:] = np.cumsum(size)
    for per in sorted({1024, max(1024, int(start[-1]) // 8192 + 1), int(start[-1]) + 1}):
        longest = lib.longest_sweep_share(start.ctypes.data_as(ctypes.c_void_p), ctypes.c_uint32(len(size)), ctypes.c_uint32(per))
        assert 0 <= longest <= per, (name, per, longest)


def test_a_chunks_long_blocks_take_more_workgroups(lib):
    for few, many in ((1, 1), (16, 32), (128, 256), (5, 5)):
        for groups in (0, 7, 100_000, 1_000_000, 10_000_000):
            shares = lib.chunk_shares(ctypes.c_uint32(groups), ctypes.c_uint32(few), ctypes.c_uint32(many))
            assert few <= shares <= many
            assert shares == many or groups < (shares + 8) * 16384
            assert shares % 8 == 0 or few % 8

"""The edge chunks' forms for devices without much memory, against the oracle bit for bit: estimates that are all doubles (in the
caller's array, or in scratch).  A process of its own loads an allocator that refuses
large requests before the library."""
import os
import subprocess
import sys
import textwrap

import pytest

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))

BODY = """
    import ctypes, sys
    refuse = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    import numpy as np, torch
    import oracle
    from paper_2502_17846_amd import binding as B
    from tests.test_gpu_edge_stream_binned import _stream
    DEV = "cuda:0"

    def stream(n, m, c_size, mode, hub, limits, refusals):
        src, dst = _stream(n, m, n % 89, hub=hub)
        if hub: src[::5] = 100_000 + src[::5] % 50_000            # blocks with most of their nodes in every chunk
        seed = (np.arange(n) % 3 == 0).astype(np.int32)
        P = n // 2 + 40
        want = oracle.edge_stream_bipartition(src, dst, n, c_size, P, seed, mode, return_state=True)
        s, d, sd = (torch.as_tensor(a).to(DEV) for a in (src, dst, seed))
        for counts, limit in zip((True, False), limits):
            refuse.refuse_above(ctypes.c_size_t(limit))
            parts, sizes, est = B.grem_edge_stream_bipartition(s, d, n, c_size, P, sd, mode, want_nbr_counts=counts)
            torch.cuda.synchronize()
            print("[case]", n, m, c_size, mode, counts, limit, refuse.refused_so_far(), flush=True)
            assert refuse.refused_so_far() == refusals
            assert np.array_equal(parts.cpu().numpy(), want[0])
            assert sizes.cpu().numpy().tolist() == want[1].tolist()
            if counts: assert np.array_equal(est.cpu().numpy().view(np.uint64), want[2].view(np.uint64))

    def bisection(n, m, limit):
        src, dst = _stream(n, m, 31)
        bits = np.random.default_rng(8).integers(0, 2, (3, n), dtype=np.int32)
        want = oracle.recursive_bisection(src, dst, n, 3, 4, 1.01, bits)
        refuse.refuse_above(ctypes.c_size_t(limit))
        got = B.grem_recursive_bisection(*(torch.as_tensor(a).to(DEV) for a in (src, dst)), n, 3, 4, 1.01, torch.as_tensor(bits.reshape(-1)).to(DEV))
        print("[case] bisection", n, m, limit, refuse.refused_so_far(), flush=True)
        assert refuse.refused_so_far() == 1
        assert np.array_equal(got.cpu().numpy(), want)

    def lean(n, c_size, chunks):                 # 0.8 to 1.9 bytes per node, the pairs, 7 KB per chunk; 16 bytes per node
        base = 2 * n + 8 * c_size + 7 * 1024 * chunks
        return base, base + 16 * (n + 262_144)

    for n, m, c_size, mode, hub in ((1 << 22, 2_000_000, 300_001, B.EDGE_REFINE, 150_000), (5_000_011, 6_000_000, 1_700_001, B.EDGE_REFINE, 150_000),
                                    (5_000_011, 3_000_000, 500_000, B.EDGE_FIXED, 0), ((1 << 25) + 70_001, 3_000_000, 1_000_000, B.EDGE_REFINE, 200_000)):
        stream(n, m, c_size, mode, hub, lean(n, c_size, -(-m // c_size)), 1)
    n, m = 5_000_011, 1_500_000
    bisection(n, m, 45 * n)
    print("done", flush=True)
"""


def test_lean_forms_equal_the_oracle(tmp_path):
    shim = str(tmp_path / "librefuse.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", shim, os.path.join(HERE, "refuse_alloc.c"), "-ldl"], check=True)
    done = subprocess.run([sys.executable, "-c", textwrap.dedent(BODY), shim], cwd=os.path.dirname(HERE), capture_output=True, text=True, timeout=110)
    print(done.stdout[-3000:], flush=True)
    assert done.returncode == 0 and "done" in done.stdout, done.stdout[-2000:] + done.stderr[-2000:]

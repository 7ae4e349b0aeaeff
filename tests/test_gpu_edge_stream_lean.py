"""The edge chunks' three forms, each of which takes the place of the one before it where there is no memory for that: against the oracle bit
for bit, and against each other where bins hold several blocks of nodes (from 67M nodes on).  A process of its own
loads an allocator that refuses large requests before the library."""
import os
import subprocess
import sys
import textwrap

import pytest

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
    import ctypes, sys
    refuse = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    import numpy as np, torch
    import oracle
    from paper_2502_17846_amd import binding as B
    from tests.test_gpu_edge_stream_binned import _stream
    DEV = "cuda:0"

    def forms(f):                                # the three forms' results, and which request each was granted
        for refusals in (0, 1, 2):
            refuse.refuse_next(refusals)
            out = f()
            torch.cuda.synchronize()
            assert refuse.refused_so_far() == refusals
            print("[case]", refusals, "refused", flush=True)
            yield out
"""
ORACLE = """
    for n, m, c_size, mode, hub in ((1 << 22, 2_000_000, 300_001, B.EDGE_REFINE, 150_000), (5_000_011, 6_000_000, 1_700_001, B.EDGE_REFINE, 150_000),
                                    (5_000_011, 3_000_000, 500_000, B.EDGE_FIXED, 0), ((1 << 25) + 70_001, 3_000_000, 1_000_000, B.EDGE_REFINE, 200_000)):
        src, dst = _stream(n, m, n % 89, hub=hub)
        if hub: src[::5] = 100_000 + src[::5] % 50_000            # blocks with most of their nodes in every chunk
        seed = (np.arange(n) % 3 == 0).astype(np.int32)
        P = n // 2 + 40
        want = oracle.edge_stream_bipartition(src, dst, n, c_size, P, seed, mode, return_state=True)
        s, d, sd = (torch.as_tensor(a).to(DEV) for a in (src, dst, seed))
        for counts in (True, False):
            for parts, sizes, est in forms(lambda: B.grem_edge_stream_bipartition(s, d, n, c_size, P, sd, mode, want_nbr_counts=counts)):
                assert np.array_equal(parts.cpu().numpy(), want[0])
                assert sizes.cpu().numpy().tolist() == want[1].tolist()
                if counts: assert np.array_equal(est.cpu().numpy().view(np.uint64), want[2].view(np.uint64))
    n, m = 5_000_011, 1_500_000
    src, dst = _stream(n, m, 31)
    bits = np.random.default_rng(8).integers(0, 2, (3, n), dtype=np.int32)
    want = oracle.recursive_bisection(src, dst, n, 3, 4, 1.01, bits)
    s, d, b = (torch.as_tensor(a).to(DEV) for a in (src, dst, bits.reshape(-1)))
    for got in forms(lambda: B.grem_recursive_bisection(s, d, n, 3, 4, 1.01, b)):
        assert np.array_equal(got.cpu().numpy(), want)
    print("done", flush=True)
"""
# 2 blocks of 16,384 nodes in a bin (against the oracle too), 2 and 8 of 32,768; ranges of 2^17 and 2^18 asked nodes (2^29 nodes: the tables'
# most).  A bin that is crowded and one with most of its nodes in each chunk, both in the bin's second half
SEVERAL = """
    for n, c_size, bin in ((70_000_003, 13_000_000, 1 << 15), (140_000_003, 4_000_000, 1 << 16), ((1 << 29) + 70_001, 5_000_000, 1 << 18)):
        m = 5 * c_size // 2
        gen = torch.Generator(device=DEV).manual_seed(n % 1000)
        src, dst = (torch.randint(0, n, (m,), generator=gen, device=DEV, dtype=torch.int32) for _ in range(2))
        for first, stride, at in ((0, 8, 5), (1, c_size // 45_000, 9)):
            src[first::stride] = at * bin + bin // 2 + src[first::stride] % min(bin // 2, 30_000)
        dst[::7] = src[::7] ^ 1
        dst[::101] = src[::101]
        dst.clamp_(max=n - 1)
        seed = (torch.arange(n, device=DEV, dtype=torch.int32) % 3 == 0).to(torch.int32)
        P, first = n // 2 + 40, None
        for out in forms(lambda: B.grem_edge_stream_bipartition(src, dst, n, c_size, P, seed, B.EDGE_REFINE)):
            if first is None: first = out
            else: assert all(torch.equal(a, b) for a, b in zip(first, out))
            del out
        assert (first[0] >= 0).sum().item() > c_size
        if n < 1 << 27:
            want = oracle.edge_stream_bipartition(src.cpu().numpy(), dst.cpu().numpy(), n, c_size, P, seed.cpu().numpy(), B.EDGE_REFINE, return_state=True)
            assert np.array_equal(first[0].cpu().numpy(), want[0]) and np.array_equal(first[2].cpu().numpy().view(np.uint64), want[2].view(np.uint64))
            del want
        del first, src, dst, seed
        torch.cuda.empty_cache()
    print("done", flush=True)
"""


@pytest.mark.parametrize("body", [ORACLE, SEVERAL], ids=["oracle", "several blocks of a bin"])
def test_the_forms_are_equal(tmp_path, body):
    shim = str(tmp_path / "librefuse.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", shim, os.path.join(HERE, "refuse_alloc.c"), "-ldl"], check=True)
    done = subprocess.run([sys.executable, "-c", textwrap.dedent(PRELUDE) + textwrap.dedent(body), shim], cwd=os.path.dirname(HERE), capture_output=True, text=True,
                          timeout=110)
    print(done.stdout[-3000:], flush=True)
    assert done.returncode == 0 and "done" in done.stdout, done.stdout[-2000:] + done.stderr[-2000:]

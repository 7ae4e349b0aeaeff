"""The plain route's merged launches (histograms in tiles of LDS, admission and spill of up to 1024 tiles in a launch
each) against the oracle: numbers of partitions at the edges of their tables and label types, chunks of one ragged
tile to 1025 tiles, long rows of one part and of many, and what a run without estimates leaves out."""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_2502_17846_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _graph(n, degree, long_rows, seed):
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 2 * degree + 1, n)
    for i, d in enumerate(long_rows):
        deg[(i * 7919 + 11) % n] = d
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    return rowptr, rng.integers(0, n, rowptr[-1]).astype(np.int32)


def _check(rowptr, colidx, n, k, slack, chunk, R, seed=None, bits=64, long_row_degree=0):
    want = oracle.partition_seeded(rowptr, colidx, n, k, slack, chunk, R, seed, return_state=True)
    rp = torch.as_tensor(rowptr.astype(np.int64 if bits == 64 else np.int32)).to(DEV)
    ci = torch.as_tensor(colidx).to(DEV)
    sd = None if seed is None else torch.as_tensor(seed).to(DEV)
    opts = B.options(B.HIST_LDS, long_row_degree=long_row_degree)
    for estimates in (True, False):
        lab, sizes, est = B.grem_partition_state(rp, ci, n, k, slack, chunk, R, sd, want_estimates=estimates, options=opts)
        assert np.array_equal(lab.cpu().numpy(), want[0])
        assert sizes.cpu().numpy().tolist() == want[1].tolist()
        if estimates:
            assert np.array_equal(est.cpu().numpy().view(np.uint32), want[2])


# 64 lanes to a vertex and one, one partition, the last k of a byte and the first of two, the largest table in LDS
@pytest.mark.parametrize("k", [1, 2, 5, 63, 64, 255, 256, 257, 1024])
@pytest.mark.parametrize("seeded", [0.0, 0.3, 1.0])
def test_numbers_of_partitions(k, seeded):
    n, chunk = 9_001, 2_300                       # three tiles, the last one ragged; a chunk of fewer tiles at the end
    rowptr, colidx = _graph(n, 6, [700, 2500, 40], k)
    rng = np.random.default_rng(k + 1)
    seed = None
    if seeded:
        seed = rng.permutation(np.arange(n) % k).astype(np.int32)
        seed[rng.random(n) >= seeded] = -1
    _check(rowptr, colidx, n, k, 1.0 if k % 2 else 1.2, chunk, 2, seed, bits=32 if k % 3 else 64)


# tiles * k on both sides of the coarse table's line, 1024 tiles and one more (the other launches)
@pytest.mark.parametrize("n,chunk,k,R", [(40_000, 40_000, 300, 1), (70_000, 33_000, 512, 1), (1 << 20, 1 << 20, 16, 1),
                                         ((1 << 20) + 1, (1 << 20) + 1, 17, 1), (300_000, 262_144, 64, 0)])
def test_tiles(n, chunk, k, R):
    rowptr, colidx = _graph(n, 3, [5000], 7)
    _check(rowptr, colidx, n, k, 1.01, chunk, R)


# rows of one part and of several, all of the chunk's rows long, more long rows than the list holds
@pytest.mark.parametrize("long_rows,degree", [([8191, 8192, 16384, 16385, 60_000], 0), ([70_000, 3, 65_536, 40_000], 1000),
                                              ([300] * 1500, 50), ([300] * 2500, 2)])
def test_long_rows(long_rows, degree):
    n = 30_000
    rowptr, colidx = _graph(n, 2, long_rows, 3)
    for k, chunk in ((16, 4_096), (200, 30_000)):
        _check(rowptr, colidx, n, k, 1.05, chunk, 3, long_row_degree=degree)


# chunks counted in LDS by the prepass (64, the most), and beyond; every size that the parts can have, rows that end with one
@pytest.mark.parametrize("longest", [65_536, 1_100_000, 2_200_000])
@pytest.mark.parametrize("chunk", [469, 461])
def test_counts_of_the_chunks_long_rows(longest, chunk):
    n = 30_000
    assert -(-n // 469) == 64 and -(-n // 461) > 64
    rowptr, colidx = _graph(n, 2, [longest, 8191, 8192, 16_384, 16_385, 32_768, 32_769, 65_537], 3)
    _check(rowptr, colidx, n, 16, 1.05, chunk, 1)


def test_inside_a_workspace_of_the_advertised_size():
    n, k, chunk = 50_000, 256, 9_000
    rowptr, colidx = _graph(n, 5, [20_000, 9_000], 5)
    want = oracle.partition(rowptr, colidx, n, k, 1.05, chunk, 2)
    need = B.grem_workspace_bytes(n, k, chunk)
    ws = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
    B.grem_set_workspace(ws[:need])
    try:
        lab = B.grem_partition(torch.as_tensor(rowptr).to(DEV), torch.as_tensor(colidx).to(DEV), n, k, 1.05, chunk, 2)
        torch.cuda.synchronize()
    finally:
        B.grem_set_workspace(None)
    assert np.array_equal(lab.cpu().numpy(), want)
    assert bool((ws[need:] == 0xA5).all())


def test_many_parts_of_long_rows_are_no_slower():
    # 3000 parts in one chunk, two passes: measured 0.56 ms; 1.7 with a fence and a ticket per part
    n, k = 200_000, 8
    rng = np.random.default_rng(2)
    deg = np.full(n, 10)
    deg[rng.choice(n, 1500, replace=False)] = 20_000
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    rp = torch.as_tensor(rowptr).to(DEV)
    ci = torch.randint(0, n, (int(rowptr[-1]),), device=DEV, dtype=torch.int32)
    best = float("inf")
    for _ in range(6):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        B.grem_partition(rp, ci, n, k, 1.05, n, 1)
        torch.cuda.synchronize()
        best = min(best, 1e3 * (time.perf_counter() - t0))
    print(f"[result] {best:.2f} ms", flush=True)
    assert best <= 1.2

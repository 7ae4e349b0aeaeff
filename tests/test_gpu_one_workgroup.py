"""Runs of the plain route that one workgroup does from the first pass to the last (grem_one.hip.h), against the oracle:
sizes at the edges of its rules, every number of rows per thread, odd numbers of partitions (half-filled counter words), partitions that
fill (ranks, placements by levels), seeds, rows of thousands of entries, vertices without any, estimates kept by the caller."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17846_amd import binding as B
from tests.test_gpu_id_orders import _ms

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _graph(n, degree, seed, hubs=0):
    rng = np.random.default_rng(seed)
    deg = rng.poisson(degree, n)
    deg[rng.integers(0, n, max(1, n // 10))] = 0
    if hubs:
        deg[rng.integers(0, n, hubs)] = 3000
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    near = (np.repeat(np.arange(n), deg) + rng.integers(-40, 41, rowptr[-1])) % n          # neighbours mostly close by
    far = rng.integers(0, n, rowptr[-1])
    return rowptr, np.where(rng.random(rowptr[-1]) < 0.7, near, far).astype(np.int32)


@pytest.mark.parametrize("n,degree,k,chunk,passes,slack,seeded,hubs", [
    (1, 3, 1, 1, 0, 1.0, 0.0, 0), (5, 2, 3, 2, 2, 1.0, 0.0, 0), (1000, 8, 2, 1000, 3, 1.0, 0.0, 0), (1023, 8, 4, 1024, 2, 1.05, 0.3, 0),
    (5000, 9, 5, 1025, 2, 1.0, 0.0, 1), (20_000, 7, 3, 2049, 3, 1.001, 0.1, 2), (20_011, 3, 8, 4096, 2, 1.0, 0.0, 0), (30_000, 12, 6, 1000, 2, 1.0, 1.0, 3),
    (30_000, 5, 7, 2000, 1, 1.0, 0.0, 0), (9000, 6, 9, 1000, 2, 1.02, 0.5, 1), (9000, 5, 8, 1500, 2, 1.02, 0.5, 1), (65_534, 4, 4, 4000, 1, 1.05, 0.0, 0), (65_535, 4, 4, 4000, 1, 1.05, 0.0, 0),
    (2000, 6, 7, 2, 1, 1.0, 0.0, 0), (4100, 2, 9, 4097, 1, 1.3, 0.0, 0), (3000, 0, 6, 700, 1, 1.0, 0.0, 0), (500, 4, 2, 100, 2, 1e9, 0.0, 0)])
@pytest.mark.parametrize("bits", [32, 64])
def test_equals_the_oracle(n, degree, k, chunk, passes, slack, seeded, hubs, bits):
    rowptr, colidx = _graph(n, degree, n % 101 + k, hubs)
    rng = np.random.default_rng(k)
    seed = None
    if seeded:
        seed = (rng.permutation(n) % k).astype(np.int32)
        seed[rng.random(n) >= seeded] = -1
    want = oracle.partition_seeded(rowptr, colidx, n, k, slack, chunk, passes, seed, return_state=True)
    rp = torch.as_tensor(rowptr).to(torch.int32 if bits == 32 else torch.int64).to(DEV)
    ci = torch.as_tensor(colidx).to(DEV)
    sd = None if seed is None else torch.as_tensor(seed).to(DEV)
    lab, sizes, est = B.grem_partition_state(rp, ci, n, k, slack, chunk, passes, sd)
    assert np.array_equal(lab.cpu().numpy(), want[0])
    assert sizes.cpu().numpy().tolist() == want[1].tolist()
    assert np.array_equal(est.cpu().numpy().view(np.uint32).reshape(n, k), want[2].reshape(n, k))
    again = B.grem_partition_seeded(rp, ci, n, k, slack, chunk, passes, sd)
    assert torch.equal(lab, again)


# rows of several parts of k_one_entries, on their edges; a count of 65,535 in either half of a word, and a row too long for it
@pytest.mark.parametrize("k", [1, 2, 3, 8])
@pytest.mark.parametrize("longest", [2048, 2049, 4096, 60_001, 65_535, 65_536])
def test_long_rows(longest, k):
    n, chunk, passes = 5000, 700, 2
    rng = np.random.default_rng(longest)
    deg = rng.poisson(3, n)
    deg[[0, 699, 700, 4000, n - 1]] = longest, 2047, longest - 1, 2 * 2048 + 1, longest
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    colidx = rng.integers(0, n, rowptr[-1]).astype(np.int32)
    seed = (np.arange(n) % k).astype(np.int32)
    for row, of in ((0, 0), (n - 1, k - 1)):             # all neighbours in one partition
        colidx[rowptr[row]:rowptr[row + 1]] = rng.integers(0, (n - k) // k, longest) * k + of
    want = oracle.partition_seeded(rowptr, colidx, n, k, 1.05, chunk, passes, seed, return_state=True)
    rp, ci, sd = (torch.as_tensor(a).to(DEV) for a in (rowptr, colidx, seed))
    lab, sizes, est = B.grem_partition_state(rp, ci, n, k, 1.05, chunk, passes, sd)
    assert np.array_equal(lab.cpu().numpy(), want[0])
    assert sizes.cpu().numpy().tolist() == want[1].tolist()
    assert np.array_equal(est.cpu().numpy().view(np.uint32).reshape(n, k), want[2].reshape(n, k))


# measured, in one workgroup and in launches (which a long_row_degree asks for): 266 and 465 us, 261 and 412, 211 and 430
@pytest.mark.parametrize("rows,longest", [(3, 60_000), (200, 1000), (1, 60_000)])
def test_long_rows_are_no_slower_than_in_launches(rows, longest):
    n, k = 10_000, 2
    rng = np.random.default_rng(1)
    deg = rng.poisson(5, n)
    deg[rng.choice(n, rows, replace=False)] = longest
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    rp, ci = torch.as_tensor(rowptr).to(DEV), torch.as_tensor(rng.integers(0, n, rowptr[-1]).astype(np.int32)).to(DEV)
    took = [_ms(lambda: B.grem_partition(rp, ci, n, k, 1.05, 1024, 2, options=o), 20) for o in (B.options(), B.options(long_row_degree=16_384))]
    print(f"[result] {rows} rows of {longest}: {took} ms", flush=True)
    assert took[0] <= 1.1 * took[1]


def test_without_room_for_it_in_the_workspace():
    # (a workspace of the advertised size holds the plain route's state and not the entries beside it: the launches per chunk)
    n, k, chunk = 20_000, 4, 1024
    rowptr, colidx = _graph(n, 9, 3)
    want = oracle.partition_seeded(rowptr, colidx, n, k, 1.05, chunk, 2, None, return_state=True)[0]
    rp, ci = torch.as_tensor(rowptr).to(DEV), torch.as_tensor(colidx).to(DEV)
    ws = torch.empty(B.grem_workspace_bytes(n, k, chunk), dtype=torch.uint8, device=DEV)
    B.grem_set_workspace(ws)
    try:
        lab = B.grem_partition_seeded(rp, ci, n, k, 1.05, chunk, 2, None)
        torch.cuda.synchronize()
    finally:
        B.grem_set_workspace(None)
    assert np.array_equal(lab.cpu().numpy(), want)

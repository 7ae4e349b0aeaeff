"""The two-phase route with slices of 512, 1024 and 2048 rows (chunks of few slices are cut finer), ragged chunks and tiles,
hubs, 1, 2 and 4 admission tiles per workgroup, and seeds that leave neighbours without a label, at the numbers of
partitions where such a neighbour is told in another way, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17846_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _graph(n, degree, hubs, seed):
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 2 * degree + 1, n)
    deg[rng.integers(0, n, hubs)] = 1200
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    return rowptr, rng.integers(0, n, rowptr[-1]).astype(np.int32)


def _check(n, chunk, k, R, seeded, degree=5, hubs=40, hub_degree=1000, slack=1.05):
    rowptr, colidx = _graph(n, degree, hubs, n % 1000 + k)
    seed = None
    if seeded:
        rng = np.random.default_rng(k)
        seed = rng.permutation(np.arange(n) % k).astype(np.int32)
        seed[rng.random(n) >= seeded] = -1
    want = oracle.partition_seeded(rowptr, colidx, n, k, slack, chunk, R, seed, return_state=True)
    rp, ci = torch.as_tensor(rowptr).to(DEV), torch.as_tensor(colidx).to(DEV)
    sd = None if seed is None else torch.as_tensor(seed).to(DEV)
    with B.Plan(rp, ci, n, chunk, options=B.options(hub_degree=hub_degree, plan_max_k=max(16, k))) as plan:
        for estimates in (True, False):         # (the admission works the hubs out itself when they are not asked for)
            need = plan.call_bytes(k, R, seeded=seed is not None, with_estimates_out=estimates)
            ws = torch.full((need + 4096,), 0xA5, dtype=torch.uint8, device=DEV)
            B.grem_set_workspace(ws[:need])
            try:
                lab, sizes, est = B.grem_partition_planned(plan, k, slack, R, sd, want_sizes=True, want_estimates=estimates)
                torch.cuda.synchronize()
            finally:
                B.grem_set_workspace(None)
            assert np.array_equal(lab.cpu().numpy(), want[0])
            assert sizes.cpu().numpy().tolist() == want[1].tolist()
            if estimates:
                assert np.array_equal(est.cpu().numpy().view(np.uint32), want[2])
            assert bool((ws[need:] == 0xA5).all())
        if seed is not None:
            counts = B.grem_plan_neighbour_counts(plan, k, sd)
            assert np.array_equal(counts.cpu().numpy(), oracle.neighbour_counts(rowptr, colidx, n, seed, k))


# rows per slice: 512 (an odd number of them in the last tile), 512 in two tiles' worth, 1024, 2048
@pytest.mark.parametrize("n,chunk", [(140_000, 67_301), (300_001, 262_144), (530_000, 522_000), (700_000, 620_001)])
@pytest.mark.parametrize("k", [6, 16, 32])
def test_slices(n, chunk, k):
    _check(n, chunk, k, 1, 0.0)


@pytest.mark.parametrize("k", [2, 8, 12, 15, 16, 17, 28, 31, 32])
@pytest.mark.parametrize("seeded", [0.1, 0.9])
def test_neighbours_without_a_label(k, seeded):
    _check(60_001, 20_000, k, 2, seeded)


def test_every_row_a_hub_and_32_bit_estimates():
    _check(30_000, 15_000, 31, 3, 0.3, degree=8, hubs=0, hub_degree=1)
    _check(140_000, 70_000, 32, 4, 0.3, hub_degree=8192)


# more than 256 and more than 512 admission tiles
@pytest.mark.parametrize("n", [400_000, 600_000])
def test_tiles_per_workgroup(n):
    _check(n, n, 16, 1, 0.2, degree=3)

"""The re-layout's units at the sizes where they change form: parts without and with empty rows, rows that begin at every
64th entry, units of exactly 8,192 entries, one less and one more (one round and two), hub rows left out, chunks whose
blocks do not tile the ids, hub shares; against the oracle's neighbour counts and partition."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17846_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N = 70_000


def _degrees(form):
    rng = np.random.default_rng(7)
    if form == "even":                       # every row begins at a multiple of 64: parts of 256 rows hold 16,384 entries
        return np.full(N, 64)
    if form == "round":                      # 256 rows of 32 entries: one round exactly; a row less or more beside it
        deg = np.full(N, 32)
        deg[256:512:256] = 31
        deg[512:1024:256] = 33
        deg[2048::2048] += rng.integers(-1, 2, deg[2048::2048].shape[0])
        return deg
    if form == "empty":                      # most rows empty, the first and last of a part among them
        deg = rng.integers(0, 120, N)
        deg[rng.random(N) < 0.7] = 0
        deg[::256] = 0
        deg[255::256] = 0
        return deg
    if form == "ones":
        return np.ones(N, np.int64)
    deg = rng.integers(1, 9, N)              # hubs: left out of their parts, in shares of their own
    deg[rng.integers(0, N, 60)] = 3000
    deg[0] = deg[255] = deg[256] = deg[N - 1] = 3000
    return deg


@pytest.mark.parametrize("chunk", [1 << 16, 40_001])
@pytest.mark.parametrize("form", ["even", "round", "empty", "ones", "hubs"])
def test_units(form, chunk):
    deg = _degrees(form)
    rowptr = np.zeros(N + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    colidx = np.random.default_rng(3).integers(0, N, rowptr[-1]).astype(np.int32)
    seed = np.random.default_rng(4).integers(0, 16, N).astype(np.int32)
    rp, ci = torch.as_tensor(rowptr).to(DEV), torch.as_tensor(colidx).to(DEV)
    for bits in (rp, rp.to(torch.int32)):
        with B.Plan(bits, ci, N, chunk, options=B.options(hub_degree=1000)) as plan:
            counts = B.grem_plan_neighbour_counts(plan, 16, torch.as_tensor(seed).to(DEV))
            assert np.array_equal(counts.cpu().numpy(), oracle.neighbour_counts(rowptr, colidx, N, seed, 16))
            lab = B.grem_partition_planned(plan, 16, 1.05, 2).cpu().numpy()
    assert np.array_equal(lab, oracle.partition_seeded(rowptr, colidx, N, 16, 1.05, chunk, 2, None))

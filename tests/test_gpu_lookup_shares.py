"""Planned calls on graphs whose ids are in order of degree (the first column blocks hold most entries): runs with and without a seed
against the oracle, counts of a labelling against numpy."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17846_amd import binding as B
from tests.test_gpu_id_orders import _csr

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# chunks of more entries than 2^24 (more workgroups for their long blocks), of fewer, an odd one; labels of four and of eight bits
@pytest.mark.parametrize("n,m,chunk,k", [(2_000_000, 20_000_000, 1 << 20, 16), (2_000_000, 20_000_000, 1 << 20, 21), (300_001, 3_000_000, 1 << 16, 7),
                                         (300_001, 3_000_000, 70_001, 16), (300_001, 3_000_000, 70_001, 32)])
def test_planned_calls_in_order_of_degree(n, m, chunk, k):
    rp, ci = _csr(n, m, "by degree")
    rowptr, colidx = rp.cpu().numpy(), ci.cpu().numpy()
    rng = np.random.default_rng(k)
    labels = rng.integers(0, k, n).astype(np.int32)
    seed = (rng.permutation(n) % k).astype(np.int32)
    seed[rng.random(n) > 0.1] = -1
    with B.Plan(rp, ci, n, chunk, options=B.options(plan_max_k=k)) as plan:
        for s in (None, seed):
            want = oracle.partition_seeded(rowptr, colidx, n, k, 1.05, chunk, 1, s, return_state=True)[0]
            got = B.grem_partition_planned(plan, k, 1.05, 1, None if s is None else torch.as_tensor(s).to(DEV))
            assert np.array_equal(got.cpu().numpy(), want)
        for lab in (labels, seed):
            row = np.repeat(np.arange(n), np.diff(rowptr))
            of = lab[colidx]
            want = np.bincount(row[of >= 0] * k + of[of >= 0], minlength=n * k)
            got = B.grem_plan_neighbour_counts(plan, k, torch.as_tensor(lab).to(DEV))
            assert np.array_equal(got.cpu().numpy().reshape(-1), want)

"""Edge buckets of lists long enough for tiles of 8,192 edges (2^25 and more, with 14 or more partitions) against the oracle: last
tiles of one edge and of all but one, runs of a few edges and of whole tiles, more buckets than the sorting in LDS takes; and
lists as long with so few buckets that their tiles have 4,096 edges."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17846_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("m,k,skew", [((1 << 25) - 1, 16, False), (1 << 25, 16, False), ((1 << 25) + 1, 17, False),
                                      ((1 << 25) + 8191, 32, False), ((1 << 25) + 777, 33, False), ((1 << 25) + 64, 1, False),
                                      ((1 << 25) + 513, 12, True), ((1 << 25) + 513, 14, True)])
def test_wide_tiles(m, k, skew):
    n = 50_021
    rng = np.random.default_rng(m % 1000 + k)
    src = rng.integers(0, n, m).astype(np.int32)
    dst = rng.integers(0, n, m).astype(np.int32)
    labels = rng.integers(0, k, n).astype(np.int32)
    if skew:                                       # most of the edges in one bucket, sorted by source
        labels[rng.random(n) < 0.95] = k - 1
        src.sort()
    got = B.grem_edge_buckets(*(torch.as_tensor(x).to(DEV) for x in (src, dst)), n, torch.as_tensor(labels).to(DEV), k)
    want = oracle.edge_buckets(src, dst, labels, k)
    for g, w in zip(got, want):
        assert np.array_equal(g.cpu().numpy(), w)


# the look-ups binned by ranges of 2^16 and of 2^17 nodes, up to 16 partitions and more, with tiles of 8,192 edges
@pytest.mark.parametrize("n,m,k", [(8_400_001, (1 << 25) + 4097, 16), (8_400_001, (1 << 25) + 77, 33), ((1 << 26) + 4099, (1 << 25) + 8191, 16),
                                   ((1 << 26) + 4099, 1 << 25, 31)])
def test_wide_tiles_after_binned_look_ups(n, m, k):
    rng = np.random.default_rng(n % 1000 + k)
    src = rng.integers(0, n, m, dtype=np.int32)
    dst = rng.integers(0, n, m, dtype=np.int32)
    labels = rng.integers(0, k, n, dtype=np.int32)
    got = B.grem_edge_buckets(*(torch.as_tensor(x).to(DEV) for x in (src, dst)), n, torch.as_tensor(labels).to(DEV), k)
    want = oracle.edge_buckets(src, dst, labels, k)
    for g, w in zip(got, want):
        assert np.array_equal(g.cpu().numpy(), w)

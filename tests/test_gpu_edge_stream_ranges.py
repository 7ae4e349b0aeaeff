"""The edge-chunk path's binned runs, against the oracle bit for bit, at the places where their forms change: estimates that
outgrow their eight bytes, labels asked for range by range (ranges that end inside the last block, loops, a hub), chunks that
hold most nodes, blocks with more of a chunk's nodes than their lists hold, counts of more than 16 bits."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17846_amd import binding as B
from tests.test_gpu_edge_stream_binned import _check, _stream

pytestmark = pytest.mark.gpu


def _few(n, m, nodes, seed, star=0):
    """Edges among `nodes` nodes that are spread over all blocks, `star` of every 3000 at one of them."""
    rng = np.random.default_rng(seed)
    ids = rng.choice(n, nodes, replace=False).astype(np.int32)
    src, dst = ids[rng.integers(0, nodes, m)], ids[rng.integers(0, nodes, m)]
    src[np.arange(m) % 3000 < star] = ids[0]
    return src, dst


# a node in 70 chunks keeps 29 bits for as many halvings at most; with 1000 ends a chunk for some 20
@pytest.mark.parametrize("n", [(1 << 22) + 3, (1 << 25) + 5])
def test_estimates_that_outgrow_eight_bytes(n):
    src, dst = _few(n, 70 * 3000, 500, 3, star=1000)
    _check(src, dst, n, 3000, n // 2 + 9, (np.arange(n) // 7 & 1).astype(np.int32), B.EDGE_REFINE)


# from 2^25 nodes, and from 2^24 where a step has 2^24 ends
@pytest.mark.parametrize("n,m,c_size,mode", [((1 << 25) + 5, 700_001, 200_000, B.EDGE_REFINE), ((1 << 25) + 33_000, 3_000_000, 1_400_000, B.EDGE_FIXED),
                                             ((1 << 24) + 77, 17_000_000, 1 << 23, B.EDGE_REFINE)])
def test_labels_asked_for(n, m, c_size, mode):
    src, dst = _stream(n, m, 13, hub=150_000)
    _check(src, dst, n, c_size, n // 2 + 100, (np.arange(n) % 3 == 0).astype(np.int32), mode)


def test_a_bisection_whose_groups_ask():
    n, levels = (1 << 25) + 9, 2
    src, dst = _stream(n, 2_000_000, 31)
    bits = np.random.default_rng(8).integers(0, 2, (levels, n), dtype=np.int32)
    want = oracle.recursive_bisection(src, dst, n, levels, 3, 1.01, bits)
    got = B.grem_recursive_bisection(*(torch.as_tensor(a).to("cuda:0") for a in (src, dst)), n, levels, 3, 1.01,
                                     torch.as_tensor(bits.reshape(-1)).to("cuda:0"))
    assert np.array_equal(got.cpu().numpy(), want)


# 0.95 ends per node: a count for every node; 70,000 more in one bin: counts of 32 bits
@pytest.mark.parametrize("hub", [0, 70_000])
def test_chunks_that_hold_most_nodes(hub):
    n = (1 << 22) + 1
    src, dst = _stream(n, 4_000_000, 17, hub=hub)
    _check(src, dst, n, 2_000_000, n // 2 + 40, (np.arange(n) % 3 == 0).astype(np.int32), B.EDGE_REFINE)


# all nodes of some blocks of 16,384 in a chunk, few of the others (blocks of 32,768 from 2^23 nodes on)
@pytest.mark.parametrize("n", [5_000_011, (1 << 23) + 100])
def test_blocks_of_more_nodes_than_lists_hold(n):
    src, dst = _stream(n, 900_000, 19)
    src[::3] = 100_000 + src[::3] % 50_000
    _check(src, dst, n, 300_000, n // 2 + 40, (np.arange(n) & 1).astype(np.int32), B.EDGE_REFINE)

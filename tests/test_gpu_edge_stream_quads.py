"""The binned edge-chunk path's lists of nodes to score, against the oracle bit for bit: chunks that touch every node (a turn's
list is full each time), one node of every group of four, one of a block, the last nodes of a run that ends inside a group."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17846_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("mode", [B.EDGE_REFINE, B.EDGE_FIXED])
@pytest.mark.parametrize("step", [1, 4, 5, 32_768])
def test_nodes_of_a_chunk(step, mode):
    n = (1 << 22) + 32_768 + 7
    rng = np.random.default_rng(step)
    nodes = np.arange(3 % step, n, step)
    nodes = np.concatenate([nodes, [n - 1, n - 2]])
    rounds = []
    for _ in range(3):                             # every chunk: each of the nodes once or twice, hubs of a few hundred ends
        a = rng.permutation(nodes)
        b = rng.permutation(nodes)
        b[rng.random(b.size) < 0.001] = nodes[0]
        rounds.append((a, b))
    src = np.concatenate([a for a, _ in rounds]).astype(np.int32)
    dst = np.concatenate([b for _, b in rounds]).astype(np.int32)
    seed = rng.integers(0, 2, n).astype(np.int32)
    seed[:1000] = 1 - seed[1000:2000]
    P = n // 2 + 5000
    s, d, sd = (torch.as_tensor(x).to(DEV) for x in (src, dst, seed))
    parts, sizes, est = B.grem_edge_stream_bipartition(s, d, n, nodes.size, P, sd, mode)
    want = oracle.edge_stream_bipartition(src, dst, n, nodes.size, P, seed, mode, return_state=True)
    assert np.array_equal(parts.cpu().numpy(), want[0])
    assert sizes.cpu().numpy().tolist() == want[1].tolist()
    assert np.array_equal(est.cpu().numpy().view(np.uint64), want[2].view(np.uint64))

"""The binned edge-chunk path's lists of nodes to score, against the oracle bit for bit: chunks that touch every node (a turn's
list is full each time), one node of every group of four, one of a block, the last nodes of a run that ends inside a group; nodes
that the first chunk labels and nodes that later ones bring, known by a count or only by an end without a label."""
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


@pytest.mark.parametrize("mode", [B.EDGE_REFINE, B.EDGE_FIXED])
@pytest.mark.parametrize("step", [1, 4, 5, 32_768])
def test_nodes_that_later_chunks_bring(step, mode):
    n = (1 << 22) + 32_768 + 7
    rng = np.random.default_rng(100 + step)
    nodes = np.concatenate([np.arange(3 % step, n - 2, step), [n - 1, n - 2]])
    old, apart, late = (nodes[i::3] for i in range(3))
    c = old.size
    among = lambda x: np.resize(rng.permutation(x), c)
    chunks = [(rng.permutation(old), among(old)),                           # labelled by the seeds
              (among(apart), np.resize(rng.permutation(apart), c)),         # no end has a label: known by `seen` alone
              (among(late), rng.permutation(np.concatenate([old, apart]))[:c]),         # new nodes' ends are labelled, the others' are not
              (among(nodes), among(nodes)), (among(nodes), among(nodes))]
    src, dst = (np.concatenate([x[i] for x in chunks]).astype(np.int32) for i in range(2))
    seed = rng.integers(0, 2, n).astype(np.int32)
    P = n // 2 + 5000 if step == 1 else (n + 1) // 2
    first = oracle.edge_stream_bipartition(src[:c], dst[:c], n, c, P, seed, mode, return_state=True)
    want = oracle.edge_stream_bipartition(src, dst, n, c, P, seed, mode, return_state=True)
    # later chunks label and store: every new node of theirs, and in refinement also the first chunk's
    assert (first[0][np.concatenate([apart, late])] == -1).all() and (want[0][apart] >= 0).all()
    assert (first[2] != want[2]).any(axis=1)[late].any()
    if mode == B.EDGE_REFINE:
        assert (first[2] != want[2]).any(axis=1)[old].any() and (first[0] != want[0])[old].any()
    parts, sizes, est = B.grem_edge_stream_bipartition(*(torch.as_tensor(x).to(DEV) for x in (src, dst)), n, c, P,
                                                       torch.as_tensor(seed).to(DEV), mode)
    assert np.array_equal(parts.cpu().numpy(), want[0])
    assert sizes.cpu().numpy().tolist() == want[1].tolist()
    assert np.array_equal(est.cpu().numpy().view(np.uint64), want[2].view(np.uint64))

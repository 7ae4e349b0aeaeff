"""The edge-chunk path's admission (a lane per one, two or four words of 64 nodes, by the size of the run) and its labels of
two bits, against the oracle bit for bit: partitions that fill inside a word, inside a block and across blocks, rejected
new nodes placed by the closed form, nodes past the last whole word."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17846_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(src, dst, n, c_size, P, seed, mode):
    s, d, sd = (torch.as_tensor(a).to(DEV) for a in (src, dst, seed))
    parts, sizes, est = B.grem_edge_stream_bipartition(s, d, n, c_size, P, sd, mode)
    want = oracle.edge_stream_bipartition(src, dst, n, c_size, P, seed, mode, return_state=True)
    assert np.array_equal(parts.cpu().numpy(), want[0])
    assert sizes.cpu().numpy().tolist() == want[1].tolist()
    assert np.array_equal(est.cpu().numpy().view(np.uint64), want[2].view(np.uint64))


def _towards_one_side(n, share, side, seed):
    """Edges from a few nodes that the seed puts on one side to `share` of all others, each once: all of them want to that
    side, until it is full."""
    rng = np.random.default_rng(seed)
    hubs = 1000
    dst = (hubs + rng.permutation(n - hubs)[:int(share * n)]).astype(np.int32)
    src = rng.integers(0, hubs, dst.size).astype(np.int32)
    src[:hubs] = np.arange(hubs)
    labels = np.full(n, side, np.int32)
    labels[1] = 1 - side
    return src, dst, labels


# words per lane: 1, 2, 4 (and blocks of 1, 8 and 32 words per wave in the scoring)
@pytest.mark.parametrize("n,side", [(70_001, 0), (2_000_003, 1), (5_000_011, 0), (17_000_003, 1), (34_000_001, 0)])
def test_partitions_that_fill(n, side):
    src, dst, labels = _towards_one_side(n, 0.7, side, n % 89)
    _check(src, dst, n, src.size // 5 + 1, (n + 1) // 2 + 7, labels, B.EDGE_REFINE)


@pytest.mark.parametrize("mode", [B.EDGE_REFINE, B.EDGE_FIXED])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 1023, 1025, 4097])
def test_small_numbers_of_nodes_with_tight_capacities(n, mode):
    rng = np.random.default_rng(n)
    for slack in (0, 1, 5):
        m = 6 * n + 3
        src, dst = rng.integers(0, n, m).astype(np.int32), rng.integers(0, n, m).astype(np.int32)
        seed = (np.arange(n) & 1).astype(np.int32)
        _check(src, dst, n, n // 2 + 1, (n + 1) // 2 + slack, seed, mode)


def test_a_bisection_whose_groups_end_inside_words():
    rng = np.random.default_rng(4)
    n, m, levels = 100_003, 400_000, 4
    src, dst = rng.integers(0, n, m).astype(np.int32), rng.integers(0, n, m).astype(np.int32)
    seeds = np.stack([(np.arange(n) >> i & 1).astype(np.int32) for i in range(levels)])
    s, d, sd = (torch.as_tensor(a).to(DEV) for a in (src, dst, seeds.reshape(-1)))
    got = B.grem_recursive_bisection(s, d, n, levels, 10, 1.01, sd, B.EDGE_REFINE)
    assert np.array_equal(got.cpu().numpy(), oracle.recursive_bisection(src, dst, n, levels, 10, 1.01, seeds, B.EDGE_REFINE))


# groups side by side from the second level on, whose halves all fill: a lane per word (with fewer words than lanes), per two and
# per four words of 64 nodes
@pytest.mark.parametrize("n,levels,chunks", [(300_007, 3, 8), (17_000_003, 2, 4), (34_000_001, 2, 3)])
@pytest.mark.parametrize("mode", [B.EDGE_REFINE, B.EDGE_FIXED])
def test_bisections_whose_halves_fill(n, levels, chunks, mode):
    src, dst, _ = _towards_one_side(n, 0.9, 0, n % 89)
    rng = np.random.default_rng(n % 83)
    seeds = rng.integers(0, 2, (levels, n), dtype=np.int32)
    seeds[:, :1000] = rng.random((levels, 1000)) < 0.3                      # most of the others follow these to half 0
    got = B.grem_recursive_bisection(*(torch.as_tensor(a).to(DEV) for a in (src, dst)), n, levels, chunks, 1.0,
                                     torch.as_tensor(seeds.reshape(-1)).to(DEV), mode)
    assert np.array_equal(got.cpu().numpy(), oracle.recursive_bisection(src, dst, n, levels, chunks, 1.0, seeds, mode))

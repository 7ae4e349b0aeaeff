"""The edge-chunk path where the chunk's edge ends are binned by ranges of nodes (from 2^22 nodes on), against the
oracle bit for bit: sizes at the edges of blocks and bins, bins of more than 65,535 pairs, loops, full partitions,
both modes; the layouts of the per-node kernels below and beside it; a bisection whose groups share the launches."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17846_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _stream(n, m, seed, hub=0):
    rng = np.random.default_rng(seed)
    src = rng.integers(0, n, m).astype(np.int32)
    dst = rng.integers(0, n, m).astype(np.int32)
    dst[::7] = src[::7] ^ 1                        # close pairs: majorities to follow
    dst[::101] = src[::101]                        # loops
    src[src >= n] = n - 1
    dst[dst >= n] = n - 1
    if hub:                                        # a bin of more pairs than 16 bits count, one node of them
        src[:hub] = n - 2
        src[-hub:] = 5
    return src, dst


def _check(src, dst, n, c_size, P, seed, mode):
    s, d, sd = (torch.as_tensor(a).to(DEV) for a in (src, dst, seed))
    parts, sizes, est = B.grem_edge_stream_bipartition(s, d, n, c_size, P, sd, mode)
    want = oracle.edge_stream_bipartition(src, dst, n, c_size, P, seed, mode, return_state=True)
    assert np.array_equal(parts.cpu().numpy(), want[0])
    assert sizes.cpu().numpy().tolist() == want[1].tolist()
    assert np.array_equal(est.cpu().numpy().view(np.uint64), want[2].view(np.uint64))
    again, _, _ = B.grem_edge_stream_bipartition(s, d, n, c_size, P, sd, mode, want_sizes=False, want_nbr_counts=False)
    assert torch.equal(parts, again)


@pytest.mark.parametrize("mode", [B.EDGE_REFINE, B.EDGE_FIXED])
@pytest.mark.parametrize("n", [1 << 22, (1 << 22) + 1, 5_000_011])
def test_binned_stream_equals_the_oracle(n, mode):
    src, dst = _stream(n, 6_000_000, n % 97, hub=150_000)
    seed = (np.arange(n) % 3 == 0).astype(np.int32)
    # (a capacity that fills: rejected requests and nodes placed in the other partition)
    _check(src, dst, n, 1_700_001, n // 2 + 40, seed, mode)


# 1, 2 and 4 words per wave (movers by node), 8 and 16 (movers by word; the chunk holds too many ends for bins)
@pytest.mark.parametrize("n,m,c_size", [(1 << 20, 900_000, 250_000), ((1 << 20) + 1, 900_000, 250_000), (3_000_001, 2_500_000, 700_000),
                                        (4_400_003, 10_500_000, 9_000_000), (8_500_001, 19_000_000, 17_500_000)])
def test_words_per_wave(n, m, c_size):
    src, dst = _stream(n, m, 11)
    _check(src, dst, n, c_size, n // 2 + 1000, (np.arange(n) & 1).astype(np.int32), B.EDGE_REFINE)


def test_an_end_out_of_range_and_a_bad_seed_are_refused():
    n = (1 << 22) + 5
    src, dst = _stream(n, 300_000, 1)
    seed = (np.arange(n) & 1).astype(np.int32)
    for bad, code in ((n, B.ERR_ARG), (-1, B.ERR_ARG), (None, B.ERR_SEED)):
        d, sd = dst.copy(), seed.copy()
        if bad is None:
            sd[src[0]] = 2
        else:
            d[-1] = bad
        with pytest.raises(B.GremError) as e:
            B.grem_edge_stream_bipartition(*(torch.as_tensor(a).to(DEV) for a in (src, d)), n, 100_000, n, torch.as_tensor(sd).to(DEV))
        assert e.value.code == code


# from 2^23 nodes on an admission block is two scoring blocks, also in groups that do not begin at the first one; a capacity
# of exactly half: rejections and placements in every group
@pytest.mark.parametrize("levels,slack", [(2, 1.0), (3, 1.004)])
def test_bisection_of_groups_whose_admission_blocks_are_two_scoring_blocks(levels, slack):
    n, m = (1 << 23) + 11_003, 9_000_000
    src, dst = _stream(n, m, 29)
    bits = np.random.default_rng(6).integers(0, 2, (levels, n)).astype(np.int32)
    want = oracle.recursive_bisection(src, dst, n, levels, 3, slack, bits)
    assert np.bincount(want, minlength=1 << levels).min() % 65_536 != 0
    got = B.grem_recursive_bisection(torch.as_tensor(src).to(DEV), torch.as_tensor(dst).to(DEV), n, levels, 3, slack,
                                     torch.as_tensor(bits).to(DEV).reshape(-1))
    assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("n,levels", [(4_300_001, 2), (200_003, 5), (1500, 11)])
def test_bisection_of_groups_side_by_side(n, levels):
    # binned; groups of several blocks; more groups than nodes in a block, most of them empty, in several batches
    src, dst = _stream(n, 2 * n, 23)
    bits = np.random.default_rng(5).integers(0, 2, (levels, n)).astype(np.int32)
    slack = 1.3 if n > 10_000 else 3.0
    want = oracle.recursive_bisection(src, dst, n, levels, 6, slack, bits)
    got = B.grem_recursive_bisection(torch.as_tensor(src).to(DEV), torch.as_tensor(dst).to(DEV), n, levels, 6, slack,
                                     torch.as_tensor(bits).to(DEV).reshape(-1))
    assert np.array_equal(got.cpu().numpy(), want)

"""Edge buckets where the label look-ups are binned (from 2^23 nodes, 2^22 edges and 2e14 of their product on) and a little
below, against a stable sort of the keys from plain torch: both sizes of a bin, packed labels and bytes, ragged tiles and batches, tiles of more than 4,096 edges, and
what is refused."""
import pytest
import torch

from paper_2502_17846_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _edges(n, m, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    src = torch.randint(0, n, (m,), generator=gen, device=DEV, dtype=torch.int32)
    dst = torch.randint(0, n, (m,), generator=gen, device=DEV, dtype=torch.int32)
    dst[::5] = torch.randint(0, 300, (dst[::5].numel(),), generator=gen, device=DEV, dtype=torch.int32)   # a crowded bin
    src[::1000], dst[-1] = n - 1, n - 1
    return src, dst, gen


# the smallest of each and one edge less; a bin of 2^16 nodes cut short; bins of 2^17 nodes; two batches (16M edges), the
# last tile ragged
@pytest.mark.parametrize("n,m", [(1 << 23, 1 << 22), (8_400_001, 5_000_003), (67_200_000, 4_200_001), (9_000_000, (1 << 24) + 8195),
                                 (1 << 23, 23_841_858), (1 << 23, 23_841_857), (47_683_716, 1 << 22), (13_000_001, (1 << 24) + 8195)])
@pytest.mark.parametrize("k", [1, 16, 17, 33, 128])
def test_binned_buckets_equal_a_stable_sort(n, m, k):
    src, dst, gen = _edges(n, m, k)
    labels = torch.randint(0, k, (n,), generator=gen, device=DEV, dtype=torch.int32)
    got_s, got_d, offsets = B.grem_edge_buckets(src, dst, n, labels, k)
    key = labels[src.long()] * k + labels[dst.long()]
    order = torch.sort(key, stable=True).indices
    assert torch.equal(got_s, src[order])
    assert torch.equal(got_d, dst[order])
    want = torch.zeros(k * k + 1, dtype=torch.int64, device=DEV)
    want[1:] = torch.cumsum(torch.bincount(key, minlength=k * k), 0)
    assert torch.equal(offsets, want)


@pytest.mark.parametrize("k", [16, 40])
def test_what_is_refused(k):
    n, m = 1 << 23, 24_000_000
    src, dst, gen = _edges(n, m, 1)
    labels = torch.randint(0, k, (n,), generator=gen, device=DEV, dtype=torch.int32)
    for bad in (n, -1, 2**31 - 1):
        d = dst.clone()
        d[m // 2] = bad
        with pytest.raises(B.GremError) as e:
            B.grem_edge_buckets(src, d, n, labels, k)
        assert e.value.code == B.ERR_ARG
    for label in (k, -1):
        bad = labels.clone()
        bad[dst[7]] = label
        with pytest.raises(B.GremError) as e:
            B.grem_edge_buckets(src, dst, n, bad, k)
        assert e.value.code == B.ERR_ARG
    # a label out of range is no matter while no edge touches the node
    node = 5_000_001
    s, d = src.clone(), dst.clone()
    s[s == node], d[d == node] = 0, 0
    labels[node] = -7
    got = B.grem_edge_buckets(s, d, n, labels, k)
    labels[node] = 0
    for a, b in zip(got, B.grem_edge_buckets(s, d, n, labels, k)):
        assert torch.equal(a, b)

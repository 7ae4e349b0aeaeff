"""The walks over the CSR entries that look labels up in a packed table (grem_edge_cut, grem_expected_cut): every
width of the table and none, the parts the columns are taken in, sizes at the edges of words and tiles."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17846_amd import binding as B
from paper_2502_17846_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

SPANS = {"one label": (5, 5), "1 bit": (-1, 0), "2 bits": (-1, 2), "4 bits": (0, 15), "4 bits, negative": (-40, -25),
         "8 bits": (-1, 254), "a bit too wide": (0, 256), "all of int32": (-2**31, 2**31 - 1)}


# below and from 2^20 vertices on (packed); 8-bit tables in 1, 2 and 8 parts
@pytest.mark.parametrize("n", [(1 << 20) - 1, 1 << 20, (1 << 20) + 259, 5_000_003, 20_000_005])
@pytest.mark.parametrize("span", sorted(SPANS))
def test_edge_cut_of_labels_of_every_width(n, span):
    lo, hi = SPANS[span]
    gen = torch.Generator(device=DEV).manual_seed(n % 1000)
    deg = torch.randint(0, 4, (n,), generator=gen, device=DEV)
    deg[n // 2] = 70_001                                   # a row longer than many tiles
    deg[-1] = 5
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rowptr[1:] = torch.cumsum(deg, 0)
    nnz = int(rowptr[-1])
    colidx = torch.randint(0, n, (nnz,), generator=gen, device=DEV, dtype=torch.int32)
    colidx[-2:] = n - 1
    labels = torch.randint(lo, hi + 1, (n,), generator=gen, device=DEV).to(torch.int32)
    labels[0], labels[-1] = lo, hi                         # the span is the whole of it
    row = torch.repeat_interleave(torch.arange(n, device=DEV), deg)
    want = int((labels[row] != labels[colidx.long()]).sum())
    for rp in (rowptr, rowptr.to(torch.int32)):
        assert int(B.grem_edge_cut(rp, colidx, n, labels).item()) == want


def test_edge_cut_on_a_captured_stream():
    g = synth.rmat(20, 2, seed=3, device=DEV)
    labels = torch.randint(0, 16, (g.n,), device=DEV, dtype=torch.int32)
    want = int(B.grem_edge_cut(g.rowptr, g.colidx, g.n, labels).item())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = B.grem_edge_cut(g.rowptr, g.colidx, g.n, labels)
    for _ in range(3):
        out.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert int(out.item()) == want


# more than one tile of 256 nodes per workgroup, a ragged last word and tile
@pytest.mark.parametrize("n", [1, 15, 257, 2048 * 256 + 17, 1_300_003])
def test_expected_cut_over_several_tiles_per_workgroup(n):
    rng = np.random.default_rng(n)
    deg = rng.integers(0, 7, n)
    deg[n // 3] = 3000
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(deg, out=rowptr[1:])
    colidx = rng.integers(0, n, rowptr[-1]).astype(np.int32)
    labels = rng.integers(-1, 3, n).astype(np.int32)
    want, want_base = oracle.expected_cut(rowptr, colidx, n, labels, 0.3)
    rp, ci, lab = (torch.as_tensor(a).to(DEV) for a in (rowptr, colidx, labels))
    got, base = B.grem_expected_cut(rp, ci, n, lab, 0.3).cpu().tolist()
    assert base == want_base                               # a sum of whole numbers
    # tails: 1e-13 per term (ratios, lgamma); sums of n terms in double
    assert abs(got - want) <= 1e-11 * max(1.0, want)
    out = torch.empty(2, dtype=torch.float64, device=DEV)
    if n <= B.grem_expected_cut_noalloc_max_n():
        assert B.grem_expected_cut_noalloc(rp, ci, n, lab, 0.3, out).cpu().tolist() == [got, base]

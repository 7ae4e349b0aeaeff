"""Estimates of the plain route kept packed (more than 512 MB of them, from 128 partitions on 256 MB; tiles of 2,048 cells): rows of cells that are
no multiple of a word, one and two bytes per label, tiles with long rows in them, short last tiles, a workspace without
room for the bits.  Whole numbers: equal to the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from paper_2502_17846_amd import binding as B
from tests.test_gpu_plain_merged import _check, _graph

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,k,chunk,R,seeded", [
    (4_068_000, 33, 270_001, 1, 0.0),      # the fewest partitions; tiles of 64 rows, the last one short
    ((1 << 21) + 1, 64, 1 << 20, 2, 0.2),  # just above the line; a last chunk of one row
    (1_390_000, 97, 33_333, 2, 1.0),         # tiles of 16 rows of 97 cells: too few to be packed
    (1_390_000, 97, 70_001, 2, 1.0),         # ... and of 32: words that end inside a row
    ((1 << 21) + 1, 64, 65_504, 1, 0.0),   # the most rows that make tiles of 16 rows of 64 cells
    ((1 << 21) + 1, 64, 65_505, 1, 0.0),   # ... and the fewest that make tiles of 32
    (263_000, 256, 50_001, 3, 0.0),        # a byte per label up to the last one
    (263_000, 257, 50_000, 2, 0.3),
    (66_000, 1024, 20_003, 3, 0.0),        # four rows to a tile
])
def test_packed(n, k, chunk, R, seeded):
    rowptr, colidx = _graph(n, 5, [9000, 20_000, 70], k)
    rng = np.random.default_rng(k)
    seed = None
    if seeded:
        seed = rng.permutation(np.arange(n) % k).astype(np.int32)
        seed[rng.random(n) >= seeded] = -1
    _check(rowptr, colidx, n, k, 1.05, chunk, R, seed, bits=32 if k % 2 else 64)


def test_workspace_without_room_for_the_bits():
    n, k, chunk = 263_000, 256, 40_000
    rowptr, colidx = _graph(n, 4, [], 3)
    rp, ci = torch.as_tensor(rowptr).to(DEV), torch.as_tensor(colidx).to(DEV)
    want = oracle.partition_seeded(rowptr, colidx, n, k, 1.05, chunk, 1, None)
    whole = B.grem_workspace_bytes(n, k, chunk)
    for size in (whole, whole - n * k // 8):
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        B.grem_set_workspace(ws)
        try:
            got = B.grem_partition(rp, ci, n, k, 1.05, chunk, 1, options=B.options(B.HIST_LDS))
            torch.cuda.synchronize()
        finally:
            B.grem_set_workspace(None)
        assert np.array_equal(got.cpu().numpy(), want)

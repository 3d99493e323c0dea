"""The neighbour list at the sizes where its kernels change: rows up to and beyond the
pairs sorted in LDS, few and many atoms per cell, every pair of atoms and cells, and
scans of one block and of several; bit for bit against the oracle."""
import numpy as np
import pytest

import oracle as O
import workloads as W

from test_gpu_parity import _np

pytestmark = pytest.mark.gpu


# lattice repeats, cutoff; 256 pairs are sorted in LDS, 32768 items scanned by one block
@pytest.mark.parametrize("reps,cut,low,high", [(1, 2.0, 0, 0), (1, 8.4, 150, 256), (1, 9.0, 257, 300), (5, 8.0, 160, 180),
                                               (8, 6.9, 100, 130), (10, 9.1, 250, 300), (12, 3.5, 14, 14),
                                               (26, 2.6, 8, 8)])
def test_rows_and_order(bop, reps, cut, low, high):
    import torch
    rng = np.random.default_rng(reps)
    pos, cell = W.cubic_lattice("bcc", 2.87, reps)
    pos = W.displace(pos, cell, 0.02, rng) + rng.integers(-2, 3, (len(pos), 3)) @ cell
    ref = O.neighbours(pos, cell, cut)
    nl = bop.build_neighbours(torch.as_tensor(pos, device="cuda"), cell, cut)
    deg = np.diff(ref["row_ptr"])
    assert low <= deg.max() <= high
    for got, key in ((nl.row_ptr, "row_ptr"), (nl.nbr_j, "nbr_j"), (nl.nbr_shift, "nbr_shift"), (nl.nbr_d, "nbr_d")):
        want = np.asarray(ref[key]).reshape(_np(got).shape)
        assert np.array_equal(_np(got).view(np.uint8), want.astype(_np(got).dtype).view(np.uint8)), key
    assert np.array_equal(np.sort(_np(nl.order)), np.arange(len(pos)))

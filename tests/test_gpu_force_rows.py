"""The force passes at the row lengths where their paths change: odd and even
numbers of contracted slots in a row, rows of up to 64 and of more than 64 pair
sums (three per pair)."""
import numpy as np
import pytest

import oracle as O
import workloads as W

from test_gpu_forces import _gpu_forces

pytestmark = pytest.mark.gpu


# reps, cutoff over the lattice constant, pairs per atom (bcc shells hold 8, 6, 12, 24, 8 atoms)
@pytest.mark.parametrize("reps,cut,deg", [(3, 0.93, 8), (3, 1.2, 14), (3, 1.5, 26), (3, 1.75, 58)])
@pytest.mark.parametrize("n_max", [5, 6])
def test_forces_by_row_length(bop, reps, cut, deg, n_max):
    pos, cell = W.cubic_lattice("bcc", 2.87, reps)
    pos = W.displace(pos, cell, 0.02, W._rng(11))
    n = len(pos)
    wl = W.Workload("rows", pos, cell, np.zeros(n, np.int32), W.canonical_d_model(cut * 2.87), n_max, 200,
                    np.full(n, 6.5))
    ref, _, _ = O.forces(wl)
    scale = max(1.0, np.abs(ref).max())
    # FP64: the recursion's loss from its moments (conditioning below 1e4 at these
    # orders) on a few hundred half units; FP32 vectors: the same on theirs, where the
    # moments themselves and so the weights are FP64
    for dtype, tol in (("f64", 1e-10), ("f32", 1e-5)):
        p, _, F = _gpu_forces(bop, wl, dtype)
        assert p.plan.deg_max == deg
        assert np.abs(F - ref).max() <= tol * scale, dtype

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


@pytest.mark.parametrize("n_max", [10, 11, 18, 19, 20])
def test_weights_by_moment_count(bop, n_max):
    """Weights at the moment counts that end the kernel's forms."""
    import torch
    pos, cell = W.cubic_lattice("bcc", 2.87, 3)
    pos = W.displace(pos, cell, 0.05, W._rng(5))
    n = len(pos)
    wl = W.Workload("w", pos, cell, np.zeros(n, np.int32), W.canonical_d_model(3.5), n_max, 200, np.full(n, 6.5))
    nl = O.neighbours(pos, cell, wl.model["r_cut"])
    H_on, H = O.build_H(wl.model, wl.species, nl)
    mu = O.moments(nl, H_on, H, n_max).reshape(-1, n_max + 1)[:10]
    on = np.asarray(H_on)[:2]
    E = 0.07
    ref = lambda m: O.weights(m, n_max, 200, E, on.reshape(-1))[0]  # noqa: E731
    want = ref(mu)
    got = bop.weights(torch.as_tensor(mu.reshape(2, 5, -1), device="cuda"), torch.as_tensor(on, device="cuda"),
                      torch.tensor([E], dtype=torch.float64, device="cuda"), n_max).cpu().numpy()
    # the reference's own response to a change of the moments by 1e-10 stands for its
    # conditioning; both sides round their moments' products, some hundreds of half units
    rng = np.random.default_rng(1)
    moved = np.max([np.abs(ref(mu * (1 + 1e-10 * rng.choice([-1.0, 1.0], mu.shape))) - want) for _ in range(4)], axis=0)
    tol = 1e3 * 2.0 ** -53 / 1e-10 * moved.max(0) + 1e-12 * np.abs(want).max(0)
    ok = np.isfinite(want).all(0) & (tol < 0.1 * np.abs(want).max(0) + 1e-300)
    assert ok[1:].any()
    assert np.all(np.abs(got - want).max(0)[ok] <= tol[ok])

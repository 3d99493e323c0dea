"""The FP32 and FP16 step kernels where a plan's longest row ends one of their forms:
16, 32 and 64 pairs and one more, in structures whose rows differ in length; workgroups
of every size; vectors of FP16 in rows longer than the packed form takes."""
import numpy as np
import pytest

import oracle as O
import workloads as W

from test_gpu_parity import _np

pytestmark = pytest.mark.gpu


def _disordered(longest, n_max):
    """A disordered d-band cell whose longest row has ``longest`` pairs: the cutoff lies
    between two of the distances found in it."""
    for seed in range(20):
        pos, cell = W.cubic_lattice("bcc", 2.9, 4)
        pos = W.displace(pos, cell, 0.12, W._rng(seed))
        far = O.neighbours(pos, cell, 6.5)
        d = np.sqrt((np.asarray(far["nbr_d"]).reshape(-1, 3) ** 2).sum(1))
        own = np.repeat(np.arange(len(pos)), np.diff(far["row_ptr"]))
        cuts = np.unique(d)
        lo, hi = 0, len(cuts) - 1                 # fewest distances at which some row has that many
        while lo < hi:
            mid = (lo + hi) // 2
            if np.bincount(own[d <= cuts[mid]], minlength=len(pos)).max() >= longest:
                hi = mid
            else:
                lo = mid + 1
        r_cut = 0.5 * (cuts[lo] + cuts[lo + 1]) if lo + 1 < len(cuts) else cuts[lo] + 1e-3
        if np.bincount(own[d < r_cut], minlength=len(pos)).max() == longest:
            n = len(pos)
            return W.Workload("rows", pos, cell, np.zeros(n, np.int32), W.canonical_d_model(float(r_cut)), n_max, 200,
                              np.full(n, 4.5))
    raise AssertionError("no such cell")


@pytest.mark.parametrize("longest,threads", [(16, 512), (17, 256), (17, 512), (32, 512), (33, 256), (33, 512), (33, 1024),
                                             (63, 512), (64, 1024), (64, 512)])
def test_step_by_longest_row(bop, longest, threads):
    n_max = 6
    wl = _disordered(longest, n_max)
    ref = O.energy_pipeline(wl)
    rp, no = np.asarray(ref["nl"]["row_ptr"]), 5
    H = np.asarray(ref["H_bond"]).reshape(-1, no, no)
    row = np.add.reduceat(np.abs(H).sum(2), rp[:-1], axis=0) + np.abs(np.asarray(ref["H_on"]))
    tuning = {"block_threads": threads}
    # a moment is n products of rows of longest * 5 + 1 terms, each rounded to a half unit
    p = bop.EnergyPath(wl.pos, wl.cell, wl.species, wl.model, n_max, 200, "f32", tuning=tuning)
    assert p.plan.deg_max == longest and p.plan.block_threads == threads
    mu = _np(p.run_moments())
    for n in range(n_max + 1):
        tol = (n + 1) * (longest * no + 4) * 2.0 ** -24 * row.max() ** n
        assert np.abs(mu[:, :, n] - ref["mu"][:, :, n]).max() <= tol, n
    # recursion coefficients: a few half units of the largest one at each of the levels
    rec = ref["rec"]
    top = max(np.abs(rec["a"]).max(), np.abs(rec["b"]).max())
    for dtype, u in (("f32", 2.0 ** -24), ("f16", 2.0 ** -11)):
        p = bop.EnergyPath(wl.pos, wl.cell, wl.species, wl.model, n_max, 200, dtype, tuning=tuning, method="lanczos")
        p.run_moments()
        for key in ("a", "b"):
            np.testing.assert_allclose(_np(p.rec[key]), rec[key], atol=8 * n_max * u * top, rtol=0)

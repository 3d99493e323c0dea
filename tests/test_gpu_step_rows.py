"""The FP32 and FP64 step kernels at the row lengths where their paths change: d
rows of up to 16 pairs (blocks through LDS) and longer ones, rows beyond the
slots held from a row ahead, s,p,d rows; FP32, FP16 and FP64 vectors."""
import numpy as np
import pytest

import oracle as O
import workloads as W

from test_gpu_parity import _np

pytestmark = pytest.mark.gpu

# lattice, orbitals, cutoff over the lattice constant: bcc shells hold 8, 6, 12, 24, 8 atoms, fcc 12, 6, 24
ROWS = [("bcc", 5, 0.93, 8), ("bcc", 5, 1.2, 14), ("bcc", 5, 1.5, 26), ("bcc", 5, 1.75, 58),
        ("fcc", 9, 0.85, 12), ("fcc", 9, 1.1, 18), ("fcc", 9, 1.3, 42)]


def _wl(kind, no, cut, n_max):
    a = 2.9 if kind == "bcc" else 3.6
    pos, cell = W.cubic_lattice(kind, a, 4 if kind == "bcc" else 3)
    pos = W.displace(pos, cell, 0.01, W._rng(7))
    model = W.canonical_d_model(cut * a) if no == 5 else W.spd_alloy_model(r_cut=cut * a)
    n = len(pos)
    spc = (np.arange(n) % model["n_species"]).astype(np.int32)
    return W.Workload("rows", pos, cell, spc, model, n_max, 200, np.full(n, 4.5))


@pytest.mark.parametrize("kind,no,cut,deg", ROWS)
@pytest.mark.parametrize("n_max", [5, 6])
def test_moments_by_row_length(bop, kind, no, cut, deg, n_max):
    wl = _wl(kind, no, cut, n_max)
    ref = O.energy_pipeline(wl)
    # |H|^n by the largest row sum; a moment is n products of rows of deg * no + 1
    # terms, each rounded to a relative half unit of the vectors' type
    H, nl = np.asarray(ref["H_bond"]), ref["nl"]
    rp = np.asarray(nl["row_ptr"])
    row = np.add.reduceat(np.abs(H.reshape(-1, no, no)).sum(2), rp[:-1], axis=0) + np.abs(np.asarray(ref["H_on"]))
    for dtype, u in (("f32", 2.0 ** -24), ("f64", 2.0 ** -53)):
        p = bop.EnergyPath(wl.pos, wl.cell, wl.species, wl.model, n_max, 200, dtype)
        assert p.plan.deg_max == deg
        mu = _np(p.run_moments())
        for n in range(n_max + 1):
            tol = (n + 1) * (deg * no + 4) * u * row.max() ** n
            assert np.abs(mu[:, :, n] - ref["mu"][:, :, n]).max() <= tol, (dtype, n)


@pytest.mark.parametrize("kind,no,cut,deg", ROWS)
@pytest.mark.parametrize("n_max", [5, 6])
def test_lanczos_by_row_length(bop, kind, no, cut, deg, n_max):
    wl = _wl(kind, no, cut, n_max)
    ref = O.energy_pipeline(wl)["rec"]
    # FP64: the reference's own loss on the way from its moments; FP32 and FP16
    # vectors: a few half units of the largest coefficient at each of the levels
    top = max(np.abs(ref["a"]).max(), np.abs(ref["b"]).max())
    for dtype, tol in (("f64", 1e-9), ("f32", 8 * n_max * 2.0 ** -24 * top), ("f16", 8 * n_max * 2.0 ** -11 * top)):
        p = bop.EnergyPath(wl.pos, wl.cell, wl.species, wl.model, n_max, 200, dtype, method="lanczos")
        p.run_moments()
        np.testing.assert_allclose(_np(p.rec["a"]), ref["a"], atol=tol, rtol=0)
        np.testing.assert_allclose(_np(p.rec["b"]), ref["b"], atol=tol, rtol=0)

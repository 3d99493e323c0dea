"""The expansion, Fermi search and energy sums at the numbers of rows and terms where
their kernels change: rows at the edges of a row block and of the search's and the
expansion's forms, terms at the edges of what is held at once, levels at the edge of
the lanes of a row; and a workspace without room for the search's own partials."""
import numpy as np
import pytest

import oracle as O

from test_gpu_parity import _np

pytestmark = pytest.mark.gpu

# atoms, orbitals, moments, terms; 65536 rows end a form of the search (16384 too, and by terms fewer than 65536:
# test_gpu_level_routes.py), 98304 one of the expansion, 8192 are one tree of its sums
CASES = [(1, 1, 3, 1), (33, 1, 20, 201), (32, 5, 21, 200), (1024, 1, 8, 202), (205, 5, 9, 203), (910, 9, 8, 51),
         (8192, 1, 6, 26), (8193, 1, 5, 52), (65536, 1, 4, 24), (65537, 1, 4, 24), (98304, 1, 6, 8), (98305, 1, 6, 8),
         (5, 9, 7, 3), (32, 2, 9, 404), (8, 5, 9, 1024)]


def _rows(n_atoms, no, n_max, seed=3):
    """Random chains (a, b), terminators and the chains' moments."""
    rng = np.random.default_rng(seed)
    R, na, nb = n_atoms * no, O.n_a(n_max), O.n_b(n_max)
    a, b = rng.uniform(-0.6, 0.6, (R, na)), rng.uniform(0.9, 1.5, (R, nb + 1))
    b[:, 0] = 0.0
    mu, v = np.zeros((R, n_max + 1)), np.zeros((R, na + nb + 3))
    v[:, 0] = 1.0
    for n in range(n_max + 1):                    # mu_n = <0|T^n|0>
        mu[:, n] = v[:, 0]
        w = np.zeros_like(v)
        w[:, :na] += a * v[:, :na]
        w[:, :nb] += b[:, 1:] * v[:, 1:nb + 1]
        w[:, 1:nb + 1] += b[:, 1:] * v[:, :nb]
        v = w
    # terminators wider than every chain, so that no state leaves the band
    rec = {"a": a, "b": b, "a_inf": rng.uniform(-0.1, 0.1, R), "b_inf": rng.uniform(2.0, 2.2, R),
           "flags": np.zeros(R, np.int32)}
    return mu, rec, rng.uniform(-0.5, 0.5, (n_atoms, no))


def _gpu(bop, mu, rec, on, n_elec, n_max, n_exp, ws=None):
    import torch
    d = lambda x: torch.as_tensor(np.ascontiguousarray(x), device="cuda")  # noqa: E731
    r = {k: d(v) for k, v in rec.items()}
    out = bop.energy(None if mu is None else d(mu), r, d(on), n_elec, n_max, n_exp, ws=ws)
    return {k: _np(v) for k, v in out.items()}


@pytest.mark.parametrize("n_atoms,no,n_max,n_exp", CASES)
def test_tail_by_rows(bop, n_atoms, no, n_max, n_exp):
    mu, rec, on = _rows(n_atoms, no, n_max)
    gs, chain = O.dos_coeffs(mu, rec, n_max, n_exp, with_chain=True)
    if n_max >= 16:                               # from the chain alone: the moments of so many are ill-conditioned
        mu = None
        m = min(n_max, n_exp) + 1
        gs[:, :m] = O.jackson(n_exp)[:m] * chain[:, :m]
    n_elec = 0.74 * n_atoms * no
    E = O.fermi(gs, rec["a_inf"], rec["b_inf"], n_elec)
    ref = O.energy(gs, rec["a_inf"], rec["b_inf"], on, E)
    got = _gpu(bop, mu, rec, on, n_elec, n_max, n_exp)
    # sums of up to 1025 terms of coefficients carrying a few half units per step of
    # their recurrence: 1e-12; the level carries them over n(E_F), of the order of one
    assert abs(float(got["E_F"][0]) - E) <= 1e-10
    for k in ("N_atom", "U_atom", "dos_atom"):
        assert np.abs(got[k] - ref[k]).max() <= 1e-10 * max(1.0, np.abs(ref[k]).max()), k
    assert abs(float(got["U_total"][0]) - ref["U_total"]) <= 1e-10 * max(1.0, np.abs(ref["U_atom"]).sum())


@pytest.mark.parametrize("n_atoms,no,n_exp", [(3, 5, 40), (700, 5, 33), (3000, 5, 12)])
def test_level_without_search_workspace(bop, n_atoms, no, n_exp):
    """A workspace that holds only what the route of many rows needs gives the same
    bits: the order of the search's additions does not depend on its form."""
    import torch
    mu, rec, on = _rows(n_atoms, no, 8)
    n_elec, R = 0.74 * n_atoms * no, n_atoms * no
    up = lambda b: (b + 255) // 256 * 256  # noqa: E731
    least = up(8 * (n_exp + 1) * R) + up(8 * 15 * (2 * ((R + 255) // 256) + 1)) + 256
    full = _gpu(bop, mu, rec, on, n_elec, 8, n_exp)
    small = _gpu(bop, mu, rec, on, n_elec, 8, n_exp, ws=torch.empty(least, dtype=torch.uint8, device="cuda"))
    for k in full:
        assert np.array_equal(full[k].view(np.int64), small[k].view(np.int64)), k
    with pytest.raises(bop.BopError):
        _gpu(bop, mu, rec, on, n_elec, 8, n_exp, ws=torch.empty(least - 256, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("R", [40, 3000, 17000, 65700])
@pytest.mark.parametrize("fill", [0.0, 1e-7, 0.3, 0.5, 0.5 + 1e-4, 0.75, 1.0 - 1e-6, 1.0])
def test_level_with_gap_and_band_edges(bop, R, fill):
    """Two sets of rows with bands about [-4, -2] and [2, 4], each row's ending at energies
    of its own: levels inside a band, at band edges, in the gap, and with no
    and all electrons, where the search bisects on, by each of its routes."""
    n_exp, half = 20, R // 2
    mu, rec, on = _rows(R, 1, 5, seed=9)
    a, b = 0.2 * rec["a"], 0.2 * rec["b"]
    shift = np.where(np.arange(R) < half, -3.0, 3.0)
    rec = {"a": a + shift[:, None], "b": b, "a_inf": shift, "b_inf": np.full(R, 0.5) * np.linspace(0.99, 1.01, R),
           "flags": np.zeros(R, np.int32)}
    gs, chain = O.dos_coeffs(mu, rec, 5, n_exp, with_chain=True)
    gs[:, :6] = O.jackson(n_exp)[:6] * chain
    n_elec = 2.0 * (half * min(2 * fill, 1.0) + (R - half) * max(2 * fill - 1.0, 0.0))
    E = float(_gpu(bop, None, rec, on, n_elec, 5, n_exp)["E_F"][0])
    # half units of the counts' terms, and of the level over their slope: 1e-12 per row
    assert abs(O.count(gs, rec["a_inf"], rec["b_inf"], E) - n_elec) <= 1e-11 * R
    lo, hi = (shift - 2 * rec["b_inf"]).min(), (shift + 2 * rec["b_inf"]).max()
    assert lo <= E <= hi

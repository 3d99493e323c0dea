"""The energy sums at the numbers of rows, terms and orbitals where a row goes from four
threads to one, with blocks that are not full: against the oracle's sums at a given
level."""
import numpy as np
import pytest

import oracle as O

from test_gpu_tail_rows import _rows

pytestmark = pytest.mark.gpu


# rows are split up to 32,767, and from 160 terms on up to 249,999
@pytest.mark.parametrize("n_atoms,no,n_exp", [(32767, 1, 24), (32768, 1, 24), (16384, 2, 1), (8193, 4, 159), (8193, 4, 160),
                                              (6554, 5, 26), (4097, 8, 12), (3641, 9, 13), (3641, 9, 160), (27777, 9, 160),
                                              (27778, 9, 160), (33000, 1, 1024)])
def test_sums_by_rows(bop, n_atoms, no, n_exp):
    import torch
    n_max = 5
    _, rec, on = _rows(n_atoms, no, n_max)
    mu = np.zeros((n_atoms * no, n_max + 1))
    mu[:, 0] = 1.0
    gs, chain = O.dos_coeffs(mu, rec, n_max, n_exp, with_chain=True)
    m = min(n_max, n_exp) + 1
    gs[:, :m] = O.jackson(n_exp)[:m] * chain[:, :m]
    E = 0.21
    ref = O.energy(gs, rec["a_inf"], rec["b_inf"], on, E)
    d = lambda x: torch.as_tensor(np.ascontiguousarray(x), device="cuda")  # noqa: E731
    got = bop.energy(None, {k: d(v) for k, v in rec.items()}, d(on), 1.0, n_max, n_exp, E_F=E)
    # sums of up to 1025 terms whose coefficients carry a few half units per step of
    # their recurrence: 1e-12; the terms' factors a half unit per rotation: 1e-13
    for k in ("N_atom", "U_atom", "dos_atom"):
        assert np.abs(got[k].cpu().numpy() - ref[k]).max() <= 2e-12 * max(1.0, np.abs(ref[k]).max()) * no, k
    assert abs(float(got["U_total"].cpu()[0]) - ref["U_total"]) <= 2e-12 * max(1.0, np.abs(ref["U_atom"]).sum())

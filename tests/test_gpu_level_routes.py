"""The Fermi search at the numbers of rows and terms where its passes change form: each
block replaying the decisions (up to 16,384 rows) or a launch between the passes, rows
staged by blocks or read as they go (by rows and terms), and the sums that the decisions'
launch holds at once.  The order of the additions is the same in all, so a workspace
that leaves only the last form must give the same bits; and the oracle's level."""
import numpy as np
import pytest

import oracle as O

from test_gpu_tail_rows import _gpu, _rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,n_exp", [(16384, 10), (16384, 40), (16385, 19), (16385, 20), (24576, 20), (24577, 63), (24577, 64),
                                     (32768, 70), (32769, 70), (49152, 64), (49153, 127), (49153, 128), (65536, 130),
                                     (65537, 130)])
def test_forms_agree(bop, R, n_exp):
    import torch
    n_max = 5
    _, rec, on = _rows(R, 1, n_max)
    up = lambda b: (b + 255) // 256 * 256  # noqa: E731
    least = up(8 * (n_exp + 1) * R) + up(8 * 15 * (2 * ((R + 255) // 256) + 1)) + 256
    mu = np.zeros((R, n_max + 1))
    mu[:, 0] = 1.0
    gs, chain = O.dos_coeffs(mu, rec, n_max, n_exp, with_chain=True)
    gs[:, :n_max + 1] = O.jackson(n_exp)[:n_max + 1] * chain[:, :n_max + 1]
    # inside the bands, and at a level whose count is all but flat and is bisected throughout
    for n_elec in (0.74 * R, 2.0 * R * (1.0 - 1e-9)):
        full = _gpu(bop, None, rec, on, n_elec, n_max, n_exp)
        small = _gpu(bop, None, rec, on, n_elec, n_max, n_exp, ws=torch.empty(least, dtype=torch.uint8, device="cuda"))
        for k in full:
            assert np.array_equal(full[k].view(np.int64), small[k].view(np.int64)), k
        # half units of the counts' terms: 1e-12 per row
        assert abs(O.count(gs, rec["a_inf"], rec["b_inf"], float(full["E_F"][0])) - n_elec) <= 1e-11 * R
    E = O.fermi(gs, rec["a_inf"], rec["b_inf"], 0.74 * R)
    assert abs(float(_gpu(bop, None, rec, on, 0.74 * R, n_max, n_exp)["E_F"][0]) - E) <= 1e-10

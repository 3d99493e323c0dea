"""The Fermi level where the count passes the number of electrons more than once
within a 4096th of the band: rows whose bands are a small part of the others', with
expansions that diverge (terminators narrower than the chains), by each of the search's
routes.  The level is the one that plain bisection comes to."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


def _case(R, scale, n_exp=100, seed=5):
    """R chains, every fourth narrowed by ``scale`` about 0.3 with a terminator of 0.6 of
    the others' width; expansions from the chains alone."""
    rng = np.random.default_rng(seed)
    n_max = 5
    na, nb = O.n_a(n_max), O.n_b(n_max)
    a, b = rng.uniform(-0.6, 0.6, (40, na)), rng.uniform(0.9, 1.5, (40, nb + 1))
    a_inf, b_inf = rng.uniform(-0.1, 0.1, 40), rng.uniform(2.0, 2.2, 40)
    b[:, 0] = 0.0
    narrow = np.arange(40) % 4 == 0
    k = np.where(narrow, scale, 1.0)
    a, b = a * k[:, None] + 0.3 * narrow[:, None], b * k[:, None]
    a_inf, b_inf = a_inf * k + 0.3 * narrow, b_inf * k * np.where(narrow, 0.6, 1.0)
    pick = np.arange(R) % 40
    rec = {"a": a[pick], "b": b[pick], "a_inf": a_inf[pick], "b_inf": b_inf[pick], "flags": np.zeros(R, np.int32)}
    mu = np.zeros((40, n_max + 1))
    mu[:, 0] = 1.0
    first = {q: v[:40] for q, v in rec.items()}
    gs, chain = O.dos_coeffs(mu, first, n_max, n_exp, with_chain=True)
    gs[:, :n_max + 1] = O.jackson(n_exp)[:n_max + 1] * chain[:, :n_max + 1]
    return rec, np.ascontiguousarray(gs), first


@pytest.mark.parametrize("R", [40, 17000, 65560])
@pytest.mark.parametrize("scale", [3e-4, 1e-4])
def test_root_is_bisections(bop, R, scale):
    import torch
    n_exp = 100
    rec, gs, first = _case(R, scale, n_exp)
    d = lambda x: torch.as_tensor(np.ascontiguousarray(x), device="cuda")  # noqa: E731
    dev, on = {q: d(v) for q, v in rec.items()}, d(np.zeros((R, 1)))
    width = (first["a_inf"] + 2 * first["b_inf"]).max() - (first["a_inf"] - 2 * first["b_inf"]).min()
    several = 0
    for t in np.linspace(-1.95, 1.95, 27):
        n40 = O.count(gs, first["a_inf"], first["b_inf"], 0.3 + t * scale)
        if not 0.0 < n40 < 80.0:
            continue
        want = O.fermi(gs, first["a_inf"], first["b_inf"], n40)
        # the count at energies of the last 4096th: several roots where it falls again
        E = want + width / 4096 * np.linspace(-0.5, 0.5, 401)
        c = np.array([O.count(gs, first["a_inf"], first["b_inf"], e) for e in E])
        several += np.count_nonzero(np.diff(np.sign(c - n40))) > 1
        dev["flags"].zero_()
        got = float(bop.energy(None, dev, on, n40 * R / 40, 5, n_exp)["E_F"].cpu()[0])
        # coefficients of up to 1e4 and slopes of 1e4 per band and more: the counts' rounding
        # is 1e-12 of the counts, and moves a root by 1e-12 of the band
        assert abs(got - want) <= 1e-11 * width, (t, got, want)
    assert several >= 5


@pytest.mark.parametrize("n_max", [20, 21])
def test_root_of_a_count_that_few_rows_stretch(bop, n_max):
    """BF16 moments of so high an order: some rows' bands are a thousand times the
    others', so that a 4096th of the band holds all of most rows' states, and the count
    there rises and falls."""
    n_exp = 60
    pos, cell = W.cubic_lattice("bcc", 2.9, 4)
    pos = W.displace(pos, cell, 0.05, np.random.default_rng(1))
    model = W.canonical_d_model(3.5)
    p = bop.EnergyPath(pos, cell, np.zeros(len(pos), np.int32), model, n_max, n_exp, "bf16")
    p.run_moments()
    bop.recursion(p.mu, n_max, out=p.rec)
    rec = {k: v.cpu().numpy() for k, v in p.rec.items()}
    gs = O.dos_coeffs(p.mu.cpu().numpy().reshape(-1, n_max + 1), rec, n_max, n_exp)
    width = (rec["a_inf"] + 2 * rec["b_inf"]).max() - (rec["a_inf"] - 2 * rec["b_inf"]).min()
    assert width > 100 * np.median(4 * rec["b_inf"])
    for fill in np.linspace(0.1, 1.9, 37):
        want = O.fermi(gs, rec["a_inf"], rec["b_inf"], fill * len(gs))
        got = float(bop.energy(p.mu, p.rec, p.H_on, fill * len(gs), n_max, n_exp)["E_F"].cpu()[0])
        # the expansions of such moments carry 1e-9 of their rounding; the roots lie 0.1 apart
        assert abs(got - want) <= 1e-6, (fill, got, want)

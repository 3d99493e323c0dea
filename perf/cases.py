"""The work whose time this framework is judged by.

A case is a dict of plain values; ``prepare`` makes what a user's program holds
before the call, ``run`` is one pass through the public entry points, ``work``
counts what the path cannot do without and ``exact`` gives the same outputs in
64 bits without the library.  The systems are those of the workloads, the tests
and the benchmark (bcc canonical d band, fcc s,p,d alloy, bcc alloy with charge
neutrality, ragged batches, ferromagnetic bcc, the warm-start network), from a
hundred atoms to the size of the headline energy.
"""
import functools
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_1803_07491_amd as bop
from paper_1803_07491_amd.batch import BatchedMoments

N_EXP = 200


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _energy(name, n, dtype, method, n_max, orbitals=5, r_max=0.0):
    return {"name": name, "kind": "energy", "nx": n[0], "ny": n[1], "nz": n[2], "dtype": dtype, "method": method,
            "n_max": n_max, "orbitals": orbitals, "r_max": r_max}


def listed():
    return [
        # a small cell as in fitting and in quick checks: latency, launches and host work
        _energy("energy 128 f64", (4, 4, 4), "f64", "moments", 9),
        # the plain double-precision path on an ordinary supercell, rebuilt as in an MD step
        _energy("energy 8k f64", (16, 16, 16), "f64", "moments", 18),
        # the single-precision path on an ordinary supercell with unequal edges
        _energy("energy 32k f32", (23, 27, 26), "f32", "lanczos", 18),
        # the headline: one energy of a large cell
        _energy("energy 128k f32", (40, 40, 40), "f32", "lanczos", 18),
        # 16-bit vectors on the matrix cores
        _energy("energy 28k bf16", (24, 24, 24), "bf16", "lanczos", 18),
        # nine orbitals per atom, binary alloy
        _energy("spd alloy 7k f32", (12, 12, 12), "f32", "lanczos", 20, orbitals=9),
        # energy and forces: the step of a relaxation of a small cell, and of MD on an ordinary one
        {"name": "forces 250 f64", "kind": "forces", "nx": 5, "ny": 5, "nz": 5, "dtype": "f64", "n_max": 10},
        {"name": "forces 12k f64", "kind": "forces", "nx": 18, "ny": 18, "nz": 18, "dtype": "f64", "n_max": 18},
        # a whole charge-neutrality cycle of an alloy cell, to max|q| < 1e-4
        {"name": "scf alloy 2k f64", "kind": "scf", "nx": 10, "ny": 10, "nz": 10, "dtype": "f64", "n_max": 16},
        # many small structures of uneven size in one batch (joining, supports, moments)
        {"name": "batch 24 f32", "kind": "batch", "structures": 24, "low": 50, "high": 2000, "dtype": "f32", "n_max": 14},
        # both spin channels of a ferromagnetic cell at given moments
        {"name": "magnetic 1k f32", "kind": "magnetic", "nx": 8, "ny": 8, "nz": 8, "dtype": "f32", "method": "lanczos",
         "n_max": 16},
        # warm-start network: gradient of a minibatch and prediction for every atom of a cell
        {"name": "mlp 4096", "kind": "mlp", "batch": 4096, "rows": 32768},
    ]


def _edges(rng, low, high, per_cell):
    """Three edges (cells) of a box of about log-uniformly many atoms in [low, high]."""
    m = (math.exp(rng.uniform(math.log(low), math.log(high))) / per_cell) ** (1.0 / 3.0)
    return [max(3, int(round(m * rng.uniform(0.85, 1.15)))) for _ in range(3)]


def draw(rng):
    kind = rng.choice(["energy"] * 5 + ["spd", "forces", "forces", "scf", "batch", "magnetic", "mlp"])
    if kind == "energy":
        dtype, method = rng.choice([("f64", "moments"), ("f64", "lanczos"), ("f32", "lanczos"), ("f32", "lanczos"),
                                    ("f32", "moments"), ("bf16", "lanczos"), ("f16", "lanczos")])
        n = _edges(rng, 60, 60000 if dtype != "f64" else 30000, 2)
        r_max = 0.0
        if dtype in ("f32", "f64") and min(n) >= 10 and rng.random() < 0.2:
            r_max = rng.choice([7.0, 10.0])
        c = _energy("", n, dtype, method, rng.randint(8, 18), r_max=r_max)
    elif kind == "spd":
        dtype, method = rng.choice([("f32", "lanczos"), ("f32", "lanczos"), ("f64", "moments"), ("f64", "lanczos")])
        n = _edges(rng, 108, 9000 if dtype == "f32" else 4000, 4)
        # (from about 14 moments on, nine orbitals want the Lanczos form: their FP64 moments lose half their digits)
        c = _energy("", n, dtype, method, rng.randint(9, 20 if method == "lanczos" else 12), orbitals=9)
    else:
        c = {"kind": kind, "dtype": "f64"}
        if kind == "forces":
            c["n_max"] = rng.randint(7, 18)
            c["nx"], c["ny"], c["nz"] = _edges(rng, 60, 12000, 2)
        elif kind == "scf":
            c["n_max"] = rng.randint(9, 16)
            c["nx"], c["ny"], c["nz"] = _edges(rng, 120, 4000, 2)
        elif kind == "batch":
            c.update(structures=rng.randint(4, 40), low=50, high=rng.randint(200, 3000), n_max=rng.randint(9, 14),
                     dtype=rng.choice(["f32", "f64"]))
        elif kind == "magnetic":
            c["n_max"] = rng.randint(9, 16)
            c["dtype"], c["method"] = rng.choice([("f32", "lanczos"), ("f64", "moments")])
            c["nx"], c["ny"], c["nz"] = _edges(rng, 54, 4000, 2)
        else:
            c["batch"] = rng.randint(500, 8192)
            c["rows"] = c["batch"] + rng.randint(0, 100000)
            c["dtype"] = "f32"
    c.pop("name", None)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
BASIS = {"bcc": [[0, 0, 0], [0.5, 0.5, 0.5]], "fcc": [[0, 0, 0], [0, 0.5, 0.5], [0.5, 0, 0.5], [0.5, 0.5, 0]]}


def _lattice(kind, a, n, sigma, rng):
    """Positions and cell of a cubic lattice, displaced by N(0, sigma^2) per component and wrapped."""
    g = np.stack(np.meshgrid(*[np.arange(m) for m in n], indexing="ij"), -1).reshape(-1, 1, 3)
    pos = ((g + np.array(BASIS[kind], float)[None]).reshape(-1, 3)) * a
    edge = np.array(n, float) * a
    if sigma > 0:
        pos = pos + rng.normal(0.0, sigma, size=pos.shape)
    frac = pos / edge
    frac -= np.floor(frac)
    frac[frac >= 1.0] = 0.0
    return frac * edge, np.diag(edge)


def _d_model(r_cut, onsite=(0.0,)):
    ns = len(onsite)
    ch = {"dds": (0, -1.0, 2.48, 5.0), "ddp": (0, 4.0 / 6.0, 2.48, 5.0), "ddd": (0, -1.0 / 6.0, 2.48, 5.0)}
    return {"n_orb": 5, "n_species": ns, "r_cut": r_cut, "d_cut": 0.0, "onsite": [[0.0, 0.0, e] for e in onsite],
            "bonds": {(i, j): dict(ch) for i in range(ns) for j in range(ns)}}


def _spd_model():
    aa = {"sss": -1.2, "sps": 1.5, "sds": -0.8, "pps": 2.0, "ppp": -0.6, "pds": -1.1, "pdp": 0.5, "dds": -0.9,
          "ddp": 0.5, "ddd": -0.1}
    back = {"pss": ("sps", -1.0), "dss": ("sds", 1.0), "dps": ("pds", -1.0), "dpp": ("pdp", -1.0)}
    bonds = {}
    for pair, f in {(0, 0): 1.0, (1, 1): 0.9, (0, 1): math.sqrt(0.9), (1, 0): math.sqrt(0.9)}.items():
        ch = {k: (1, f * v, 2.5, 1.8) for k, v in aa.items()}
        ch.update({k: (1, s * f * aa[o], 2.5, 1.8) for k, (o, s) in back.items()})
        bonds[pair] = ch
    return {"n_orb": 9, "n_species": 2, "r_cut": 4.2, "d_cut": 0.0, "onsite": [[-4.0, 2.0, 0.0], [-3.5, 2.5, 0.5]],
            "bonds": bonds}


def _structure(c, seed):
    """Positions, cell, species, model and electrons per atom of a case with one cell."""
    rng = np.random.Generator(np.random.PCG64(seed))
    n = (c["nx"], c["ny"], c["nz"])
    kind = c["kind"]
    if kind == "energy" and c["orbitals"] == 9 or kind == "scf":
        fcc = kind == "energy"
        pos, cell = _lattice("fcc", 3.5355, n, 0.0, rng) if fcc else _lattice("bcc", 2.87, n, 0.0, rng)
        N = len(pos)
        spc = rng.permutation((np.arange(N) >= N // 2).astype(np.int32))
        model = _spd_model() if fcc else _d_model(3.5, (0.0, 0.8))
        return pos, cell, spc, model, np.where(spc == 0, 9.0, 8.0) if fcc else np.where(spc == 0, 6.0, 5.0)
    if kind == "magnetic":
        pos, cell = _lattice("bcc", 2.87, n, 0.03, rng)
        return pos, cell, np.zeros(len(pos), np.int32), _d_model(3.5), np.full(len(pos), 6.5)
    pos, cell = _lattice("bcc", 3.16, n, 0.08, rng)
    return pos, cell, np.zeros(len(pos), np.int32), _d_model(3.8), np.full(len(pos), 4.5)


def _ragged(c, seed):
    """Structures of uneven size, bcc or fcc at one density; the sizes belong to the case, the atoms to the seed."""
    sizes, rng = np.random.Generator(np.random.PCG64(1000 + c["structures"])), np.random.Generator(np.random.PCG64(seed))
    out = []
    for _ in range(c["structures"]):
        atoms = math.exp(sizes.uniform(math.log(c["low"]), math.log(c["high"])))
        kind = ("bcc", "fcc")[int(sizes.integers(0, 2))]
        per = len(BASIS[kind])
        m = max(2, int(round((atoms / per) ** (1.0 / 3.0))))
        pos, cell = _lattice(kind, (per / 0.085) ** (1.0 / 3.0), (m, m, m), 0.05, rng)
        out.append(SimpleNamespace(pos=pos, cell=cell, species=np.zeros(len(pos), np.int32)))
    return out


def _spins(c, seed):
    """Shifts and moments of a ferromagnetic state on its way to self-consistency."""
    rng = np.random.Generator(np.random.PCG64(seed + 1))
    n = 2 * c["nx"] * c["ny"] * c["nz"]
    return rng.normal(0.0, 0.05, n), rng.uniform(0.8, 1.8, n)


def _network(c, seed):
    """Standardised features and targets of the size and spread that the charge-neutrality cycles give."""
    rng = np.random.Generator(np.random.PCG64(seed))
    x = rng.normal(size=(c["rows"], 6)).astype(np.float32)
    t = (0.19 * np.tanh(x @ rng.normal(size=6) * 0.5)).astype(np.float32)
    return x, t


def prepare(case, seed):
    kind = case["kind"]
    s = SimpleNamespace(case=case, kind=kind)
    if kind == "batch":
        s.batch = BatchedMoments(_ragged(case, seed), _d_model(3.6), case["n_max"], dtype=case["dtype"])
    elif kind == "mlp":
        x, t = _network(case, seed)
        s.x, s.t = torch.as_tensor(x, device="cuda"), torch.as_tensor(t, device="cuda")
        s.xb, s.tb = s.x[:case["batch"]].contiguous(), s.t[:case["batch"]].contiguous()
        s.net = bop.MLP(seed=3)
    else:
        pos, cell, spc, model, val = _structure(case, seed)
        s.n_elec = float(val.sum())
        if kind == "energy":
            s.path = bop.EnergyPath(pos, cell, spc, model, case["n_max"], N_EXP, case["dtype"], method=case["method"],
                                    r_max=case["r_max"])
        elif kind == "forces":
            s.path = bop.EnergyPath(pos, cell, spc, model, case["n_max"], N_EXP, case["dtype"])
        elif kind == "scf":
            s.path = bop.SCFPath(pos, cell, spc, model, case["n_max"], val, N_EXP, case["dtype"], mixer="broyden")
            s.start = torch.zeros(len(pos), dtype=torch.float64, device="cuda")
        else:
            s.path = bop.MagneticPath(pos, cell, spc, model, case["n_max"], val, 0.8, n_exp=N_EXP, dtype=case["dtype"],
                                      method=case["method"])
            s.path.set_state(*_spins(case, seed))
    return s


def run(s):
    kind = s.kind
    if kind == "batch":
        return {"mu": s.batch.step()}
    if kind == "mlp":
        loss, g = s.net.grad(s.xb, s.tb)
        return {"loss": loss, "grad": g, "y": s.net.predict(s.x)}
    p = s.path
    if kind == "energy":
        out = p.step(s.n_elec)
        coef = {"mu": p.mu} if p.method == "moments" else {"a": p.rec["a"], "b": p.rec["b"]}
        return {**out, **coef, "flags": p.rec["flags"]}
    if kind == "forces":
        p.rebuild()
        return {**p.forces(s.n_elec), "mu": p.mu}
    if kind == "scf":
        p.set_shift(s.start)
        it, _ = p.run_scf(mix=0.5, tol=1e-4)
        return {**p.out, "shift": p.shift, "iterations": it}
    return {**p.energy(), "m_out": p.m_out, "U_X": p.U_X}


# ---------------------------------------------------------------------------
# what the path cannot do without
# ---------------------------------------------------------------------------
@functools.lru_cache(maxsize=None)
def _supports(kind, hops):
    """Atoms within k = 0..hops bonds of one atom of the perfect infinite lattice (first two shells bond)."""
    steps = ([(a, b, c) for a in (-1, 1) for b in (-1, 1) for c in (-1, 1)] if kind == "bcc" else
             [p for a in (-1, 1) for b in (-1, 1) for p in ((0, a, b), (a, 0, b), (a, b, 0))])
    steps += [tuple(2 * s * (i == j) for j in range(3)) for i in range(3) for s in (-1, 1)]
    seen, edge, out = {(0, 0, 0)}, {(0, 0, 0)}, [1]
    for _ in range(hops):
        edge = {(x + a, y + b, z + c) for x, y, z in edge for a, b, c in steps} - seen
        seen |= edge
        out.append(len(seen))
    return out, len(steps)


def _path_work(N, no, n_max, lattice, bonds=None):
    """Operations of the H.X products on the exact supports and of the tail, for N atoms."""
    K, deg = n_max // 2, bonds
    rows, d = _supports(lattice, K)
    deg = deg or d
    seen = [min(r, N) for r in rows]
    hx = no * (2 * no * no * deg + 2 * no) * (sum(seen[:K]) + (seen[K] if n_max % 2 else 0))
    tail = no * N_EXP * (5 * (n_max // 2 + 1) + 2 * 60)
    return N * (hx + tail)


def work(case):
    kind = case["kind"]
    if kind == "mlp":
        per = 2 * (6 * 64 + 64 * 64 + 64)
        return {"bytes": 4.0 * (7 * case["batch"] + 7 * case["rows"] + 2 * 4673),
                "flops": float(per * (3 * case["batch"] + case["rows"]))}
    if kind == "batch":
        N = [len(w.species) for w in _ragged(case, 0)]
        return {"bytes": float(sum(N) * (24 + 14 * 40 + 5 * 8 * (case["n_max"] + 1))),
                "flops": float(sum(_path_work(n, 5, case["n_max"], "bcc") for n in N))}
    fcc = kind == "energy" and case["orbitals"] == 9
    no, lattice = (9, "fcc") if fcc else (5, "bcc")
    N = case["nx"] * case["ny"] * case["nz"] * (4 if fcc else 2)
    out = N * (3 * 8 + no * 8 * (case["n_max"] + 1))
    flops = _path_work(N, no, case["n_max"], lattice)
    if kind == "forces":
        rows, deg = _supports(lattice, case["n_max"] // 2)
        n = case["n_max"]
        walk = sum(min(rows[min(m, n - m)], N) for m in range(1, n))
        flops += N * 5 * deg * (50 + 190) * walk
        out += N * 24
    elif kind == "scf":
        flops *= 9
    elif kind == "magnetic":
        flops *= 2
        out *= 2
    return {"bytes": float(28 * N + out), "flops": float(flops)}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _one(v):
    return torch.tensor([v], dtype=torch.float64)


def _pairs(pos, cell, r_cut):
    """All (i, j, d) with 0 < |d| < r_cut, d = r_j + S.A - r_i, ordered by (i, j, S)."""
    n = len(pos)
    reach = [int(math.ceil(r_cut / cell[k, k])) for k in range(3)]
    p = pos if isinstance(pos, torch.Tensor) else torch.as_tensor(pos, device=_device())
    q = p.detach()
    found = []
    for a in range(-reach[0], reach[0] + 1):
        for b in range(-reach[1], reach[1] + 1):
            for c in range(-reach[2], reach[2] + 1):
                S = torch.as_tensor(np.array([a, b, c], float) @ cell, device=p.device)
                near = torch.zeros((n, n), dtype=p.dtype, device=p.device)
                for x in range(3):
                    near += (q[None, :, x] + S[x] - q[:, None, x]) ** 2
                i, j = torch.nonzero((near < r_cut ** 2) & (near > 1e-12), as_tuple=True)
                found.append((i, j, S.expand(len(i), 3)))
    i, j, S = (torch.cat([f[k] for f in found]) for k in range(3))
    at = torch.argsort(i * n + j, stable=True)
    i, j, S = i[at], j[at], S[at]
    return i, j, p[j] + S - p[i]


def _blocks(model, spc, i, j, d):
    """Two-centre Slater-Koster blocks [P, no, no] along the bond vectors d, from the real harmonics and their gradients."""
    r = d.norm(dim=1)
    u = d / r[:, None]
    x, y, z = u[:, 0], u[:, 1], u[:, 2]
    o, s3 = torch.zeros_like(x), math.sqrt(3.0)
    Y = torch.stack([z * z - 0.5 * (x * x + y * y), s3 * x * z, s3 * y * z, 0.5 * s3 * (x * x - y * y), s3 * x * y], 1)
    G = torch.stack([torch.stack(g, 1) for g in ([-x, -y, 2 * z], [s3 * z, o, s3 * x], [o, s3 * z, s3 * y],
                                                [s3 * x, -s3 * y, o], [s3 * y, s3 * x, o])], 1)
    V = {}
    ns = model["n_species"]
    spc = torch.as_tensor(spc, device=d.device).long()
    for name in model["bonds"][(0, 0)]:
        tab = torch.tensor([[model["bonds"][(a, b)][name][k] for k in range(4)] for a in range(ns) for b in range(ns)],
                           dtype=d.dtype, device=d.device)[spc[i] * ns + spc[j]]
        V[name] = (tab[:, 1] * torch.where(tab[:, 0] == 0, (tab[:, 2] / r) ** tab[:, 3],
                                           torch.exp(-tab[:, 3] * (r - tab[:, 2]))))[:, None, None]
    eye5 = torch.eye(5, dtype=d.dtype, device=d.device)
    ps = Y[:, :, None] * Y[:, None, :]
    pp = (G @ G.transpose(1, 2).contiguous() - 4 * ps) / 3
    dd = V["dds"] * ps + V["ddp"] * pp + V["ddd"] * (eye5 - ps - pp)
    if model["n_orb"] == 5:
        return dd
    v = u[:, [2, 0, 1]]                               # p_z, p_x, p_y
    Gv = G[:, :, [2, 0, 1]].transpose(1, 2)           # [P, 3, 5]
    pd = v[:, :, None] * Y[:, None, :]
    pdp = (Gv - 2 * pd) / s3
    uu = v[:, :, None] * v[:, None, :]
    H = d.new_zeros((len(r), 9, 9))
    H[:, :1, :1] = V["sss"]
    H[:, :1, 1:4], H[:, 1:4, :1] = V["sps"] * v[:, None, :], V["pss"] * v[:, :, None]
    H[:, :1, 4:], H[:, 4:, :1] = V["sds"] * Y[:, None, :], V["dss"] * Y[:, :, None]
    H[:, 1:4, 1:4] = V["pps"] * uu + V["ppp"] * (torch.eye(3, dtype=d.dtype, device=d.device) - uu)
    H[:, 1:4, 4:] = V["pds"] * pd + V["pdp"] * pdp
    H[:, 4:, 1:4] = (V["dps"] * pd + V["dpp"] * pdp).transpose(1, 2)
    H[:, 4:, 4:] = dd
    return H


class _Operator:
    """H.X for X [N, no, columns], from padded neighbour slots."""

    def __init__(self, model, pos, cell, spc):
        i, j, d = _pairs(pos, cell, model["r_cut"])
        N, no = len(spc), model["n_orb"]
        deg = torch.bincount(i, minlength=N)
        first = torch.cumsum(deg, 0) - deg
        D = int(deg.max())
        slot = torch.arange(len(i), device=i.device) - first[i]
        self.nb = torch.arange(N, device=i.device)[:, None].repeat(1, D)
        self.H = d.new_zeros((N, D, no, no))
        self.nb[i, slot] = j
        self.H[i, slot] = _blocks(model, spc, i, j, d)
        lev = [0, 1, 1, 1, 2, 2, 2, 2, 2] if no == 9 else [2] * 5
        on = torch.tensor(model["onsite"], dtype=d.dtype, device=d.device)
        self.on = on[torch.as_tensor(spc, device=d.device).long()][:, lev]
        self.N, self.no, self.D = N, no, D

    def __call__(self, X, on):
        Y = on[:, :, None] * X
        for s in range(self.D):
            Y += torch.matmul(self.H[:, s].contiguous(), X[self.nb[:, s]])
        return Y


def _columns(op, on, n_max, method, keep=None):
    """Moments [R, n_max + 1] or Lanczos coefficients a [R, na], b [R, nb + 1], column block by column block."""
    R, K = op.N * op.no, n_max // 2
    step = max(op.no, int(2e8 // R) // op.no * op.no)
    parts = []
    for c0 in range(0, R, step):
        c = torch.arange(c0, min(R, c0 + step), device=on.device)
        X = on.new_zeros((op.N, op.no, len(c)))
        X[c // op.no, c % op.no, c - c0] = 1.0
        mask = None if keep is None else keep[:, c // op.no][:, None, :]
        apply = (lambda Z: op(Z, on)) if mask is None else (lambda Z: op(Z, on) * mask)
        dot = lambda P, Q: (P * Q).sum((0, 1))  # noqa: E731
        if method == "moments":
            mu = [torch.ones_like(X[0, 0])]
            for _ in range(K):
                Z = apply(X)
                mu += [dot(X, Z), dot(Z, Z)]
                X = Z
            if n_max % 2:
                mu.append(dot(X, apply(X)))
            parts.append(torch.stack(mu, 1))
            continue
        a, b, old = [], [torch.zeros_like(X[0, 0])], torch.zeros_like(X)
        for k in range(K + n_max % 2):
            Z = apply(X) - b[-1] * old
            a.append(dot(X, Z))
            if k < K:
                Z -= a[-1] * X
                b.append(dot(Z, Z).sqrt())
                old, X = X, Z / b[-1]
        parts.append(torch.cat([torch.stack(a, 1), torch.stack(b, 1)], 1))
    return torch.cat(parts)


def _chain_energy(a, b, e_on, n_elec):
    """E_F and per-row N, U, n(E_F) (one spin) of terminated chains; rows in blocks of the sums' size."""
    R, na, nb = len(a), a.shape[1], b.shape[1] - 1
    up = torch.zeros_like(a)
    up[:, :min(na, nb)] = b[:, 1:1 + min(na, nb)]
    low = b[:, :na]
    lo, hi = (a - low - up).min(1).values, (a + low + up).max(1).values
    A, B = 0.5 * (hi + lo), 0.25 * (hi - lo)
    L = N_EXP + 2
    ah, bh = a.new_zeros((R, L)), a.new_full((R, L + 1), 0.5)
    ah[:, :na] = (a - A[:, None]) / (2 * B)[:, None]
    bh[:, 0] = 0.0
    bh[:, 1:nb + 1] = b[:, 1:] / (2 * B)[:, None]
    z0, z1 = torch.zeros_like(ah), torch.zeros_like(ah)
    z1[:, 0] = 1.0
    sig = [z1[:, 0]]
    for _ in range(N_EXP):
        z2 = 2 * ah * z1 - z0
        z2[:, 1:] = z2[:, 1:] + 2 * bh[:, 1:L] * z1[:, :-1]
        z2[:, :-1] = z2[:, :-1] + 2 * bh[:, 1:L] * z1[:, 1:]
        z0, z1 = z1, z2
        sig.append(z1[:, 0])
    m = torch.arange(N_EXP + 1, dtype=a.dtype, device=a.device)
    w = math.pi / (N_EXP + 1)
    g = ((N_EXP - m) * torch.cos(w * (m + 1)) + torch.sin(w * (m + 1)) / math.tan(w)) / (N_EXP + 1)
    gs = (g / g[0]) * torch.stack(sig, 1)

    def sums(E, count_only=False):
        c = ((E - A) / (2 * B)).clamp(-1.0, 1.0)
        phi = torch.arccos(c)[:, None]
        k = torch.arange(1, N_EXP + 4, dtype=a.dtype, device=a.device)
        sk = torch.sin(k * phi) / k
        chi = torch.cat([1 - phi / math.pi + sk[:, 1:2] / math.pi, (sk[:, 2:] - sk[:, :-2]) / math.pi], 1)
        N = (gs * chi[:, :N_EXP + 1]).sum(1)
        if count_only:
            return N
        U = (gs[:, :N_EXP] * chi[:, 1:N_EXP + 1]).sum(1) + (gs[:, 1:] * chi[:, :N_EXP]).sum(1)
        U = U + gs[:, N_EXP] * chi[:, N_EXP + 1]
        D = (gs * sk[:, :N_EXP + 1] * k[:N_EXP + 1]).sum(1) / (math.pi * B)
        return N, B * U + (A - e_on) * N, torch.where(c.abs() < 1, D, torch.zeros_like(D))

    with torch.no_grad():
        x0, x1 = float((A - 2 * B).min()), float((A + 2 * B).max())
        for _ in range(64):
            E = 0.5 * (x0 + x1)
            if E <= x0 or E >= x1:
                break
            if float(sums(E, True).sum()) < n_elec:
                x0 = E
            else:
                x1 = E
    return 0.5 * (x0 + x1), sums


def _tail(coef, on, n_max, n_elec, spin=2.0):
    """E_F and per-atom N, U, n(E_F) from Lanczos coefficients [R, na + nb + 1]; n_elec counts `spin` per state."""
    na = (n_max - 1) // 2 + 1
    E, sums = _chain_energy(coef[:, :na], coef[:, na:], on.reshape(-1), n_elec / spin)
    N, U, D = (spin * v.reshape(on.shape).sum(1) for v in sums(E))
    return E, N, U, D


def _cycle(op, case, val):
    """Broyden charge-neutrality cycle from zero shifts, as documented for SCFPath (mix 0.5, floor 1e-3, tolerance 1e-4)."""
    n0 = torch.as_tensor(val, device=op.on.device)
    x, mix, H, last = torch.zeros_like(n0), 0.5, [], None
    for it in range(1, 60):
        on = op.on + x[:, None]
        E, N, U, D = _tail(_columns(op, on, case["n_max"], "lanczos"), on, case["n_max"], float(val.sum()))
        q = N - n0
        if float(q.abs().max()) < 1e-4:
            return {"E_F": _one(E), "N_atom": N, "U_atom": U, "dos_atom": D, "U_total": U.sum().reshape(1), "shift": x,
                    "iterations": it}
        F = q / D.clamp(min=1e-3)
        back = lambda v: -mix * v + sum((u * torch.dot(w, v) for u, w in H), torch.zeros_like(v))  # noqa: E731
        if last is not None:
            s, y = x - last[0], F - last[1]
            H.append(((s - back(y)) / torch.dot(y, y), y))
        last = (x, F)
        x = x - back(F)
        x = x - x.mean()
    return None


def _forces(model, pos, cell, spc, case, n_elec):
    """Energy and -dU/dr at fixed electron count, by differentiating dense powers of H."""
    dev = _device()
    r = torch.tensor(pos, device=dev, requires_grad=True)
    N, n = len(spc), case["n_max"]
    i, j, d = _pairs(r, cell, model["r_cut"])
    H = torch.zeros((N, N, 5, 5), dtype=torch.float64, device=dev).index_put((i, j), _blocks(model, spc, i, j, d), True)
    H = H.permute(0, 2, 1, 3).reshape(5 * N, 5 * N)
    powers = [torch.eye(5 * N, dtype=torch.float64, device=dev)]
    for _ in range((n + 1) // 2):
        powers.append(powers[-1] @ H)
    mu = torch.stack([(powers[(k + 1) // 2] * powers[k // 2]).sum(1) for k in range(n + 1)], 1)
    # recursion coefficients from the moments: orthonormal polynomials by their coefficients in powers of H
    na, nb = (n - 1) // 2 + 1, n // 2
    R, zero = 5 * N, torch.zeros(5 * N, dtype=torch.float64, device=dev)
    pair = lambda p, q, o: sum(p[k] * q[l] * mu[:, k + l + o] for k in range(len(p)) for l in range(len(q)))  # noqa: E731
    a, b, old, cur = [], [zero], [], [torch.ones_like(zero)]
    for k in range(na):
        a.append(pair(cur, cur, 1))
        if k + 1 > nb:
            break
        nxt = [zero] + cur
        nxt = [v - (a[-1] * cur[t] if t < len(cur) else 0) - (b[-1] * old[t] if t < len(old) else 0)
               for t, v in enumerate(nxt)]
        b.append(pair(nxt, nxt, 0).sqrt())
        old, cur = cur, [v / b[-1] for v in nxt]
    e = torch.zeros(R, dtype=torch.float64, device=dev)
    E, sums = _chain_energy(torch.stack(a, 1), torch.stack(b, 1), e, n_elec / 2)
    Nr, Ur, Dr = sums(E)
    Eb = float((e * Dr.detach()).sum() / Dr.detach().sum())
    F = -torch.autograd.grad(2 * (Ur.sum() - (E - Eb) * Nr.sum()), r)[0]
    per = lambda v: 2 * v.detach().reshape(N, 5).sum(1)  # noqa: E731
    return {"E_F": _one(E), "N_atom": per(Nr), "U_atom": per(Ur), "dos_atom": per(Dr),
            "U_total": per(Ur).sum().reshape(1), "F": F, "mu": mu.detach().reshape(N, 5, n + 1)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "mlp":
        x, t = (torch.as_tensor(v, device=_device()).double() for v in _network(case, seed))
        flat = bop.MLP(seed=3, device="cpu").params.double().to(x.device)
        parts, o = [], 0
        for shape in ((64, 6), (64,), (64, 64), (64,), (1, 64), (1,)):
            k = math.prod(shape)
            parts.append(flat[o:o + k].reshape(shape).clone().requires_grad_())
            o += k
        net = lambda v: (torch.tanh(torch.tanh(v @ parts[0].T + parts[1]) @ parts[2].T + parts[3]) @ parts[4].T  # noqa: E731
                         + parts[5])[:, 0]
        B = case["batch"]
        loss = ((net(x[:B]) - t[:B]) ** 2).mean()
        g = torch.cat([v.reshape(-1) for v in torch.autograd.grad(loss, parts)])
        return {"loss": loss.detach().reshape(1), "grad": g, "y": net(x).detach()}
    with torch.no_grad():
        if kind == "batch":
            every = _ragged(case, seed)
            if sum(len(w.species) ** 2 for w in every) > 1.5e8:
                return None
            mu = []
            for w in every:
                op = _Operator(_d_model(3.6), w.pos, w.cell, w.species)
                mu.append(_columns(op, op.on, case["n_max"], "moments").reshape(op.N, 5, -1))
            return {"mu": torch.cat(mu)}
        pos, cell, spc, model, val = _structure(case, seed)
        N, n_max = len(pos), case["n_max"]
        if kind == "forces":
            if N > 700 or n_max > 12:                 # dense powers; beyond, the moments' own recursion loses digits
                return None
            with torch.enable_grad():
                return _forces(model, pos, cell, spc, case, float(val.sum()))
        if N > (700 if kind == "scf" else 2500 if kind == "energy" and case["orbitals"] == 9 else 8500):
            return None
        op = _Operator(model, pos, cell, spc)
        if kind == "scf":
            return _cycle(op, case, val)
        if kind == "magnetic":
            shift, m = (torch.as_tensor(v, device=op.on.device) for v in _spins(case, seed))
            ons = [op.on + (shift - s * 0.4 * m)[:, None] for s in (1.0, -1.0)]
            coef = torch.cat([_columns(op, on, n_max, "lanczos") for on in ons])
            E, Nv, U, D = _tail(coef, torch.cat(ons), n_max, float(val.sum()), spin=1.0)
            m_out = Nv[:N] - Nv[N:]
            return {"E_F": _one(E), "N_atom": Nv, "U_atom": U, "dos_atom": D, "U_total": U.sum().reshape(1),
                    "m_out": m_out, "U_X": (-0.25 * 0.8 * (m_out ** 2).sum()).reshape(1)}
        keep = None
        if case["r_max"] > 0:
            p, edge = torch.as_tensor(pos, device=op.on.device), torch.as_tensor(np.diag(cell).copy(), device=op.on.device)
            far = torch.zeros((N, N), dtype=torch.float64, device=op.on.device)
            for x in range(3):
                d = p[:, None, x] - p[None, :, x]
                far += (d - edge[x] * torch.round(d / edge[x])) ** 2
            keep = (far <= case["r_max"] ** 2).double()
        coef = _columns(op, op.on, n_max, "lanczos", keep)
        E, Na, U, D = _tail(coef, op.on, n_max, float(val.sum()))
        out = {"E_F": _one(E), "N_atom": Na, "U_atom": U, "dos_atom": D, "U_total": U.sum().reshape(1)}
        if case["method"] == "moments":
            out["mu"] = _columns(op, op.on, n_max, "moments", keep).reshape(N, op.no, -1)
        else:
            na = (n_max - 1) // 2 + 1
            out["a"], out["b"] = coef[:, :na], coef[:, na:]
        return out

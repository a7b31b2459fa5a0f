"""The calls whose speed matters to a user of this framework, with their inputs and 64-bit values.

listed() names the cases, draw() gives others of the same ranges, prepare() makes what a program has in hand before
the call (positions, a model handle, a neighbour list, coefficients, a network), run() is one pass through the public
entry points, work() the bytes and operations that the pass cannot do without, and exact() the values that run()
returns, from plain torch in 64 bits (the defining formulas of the descriptors, none of this repository's code).

Inputs are tantalum-like lattices with displaced atoms and vacancies, as in the molecular-dynamics boxes and the
training cells of the framework's workloads.  Coefficients give the 2-, 3- and 4-body energies of an atom spreads
of about 1, 0.3 and 0.1 eV.  E, W and G of an FP32 handle are totals in double of values that hold FP32 digits, and
are returned in the handle's type.
"""
import itertools
import math

import numpy as np
import torch

from paper_2212_14446_amd import autograd, md, pod, surrogate

DEV = "cuda"
A0 = 3.31                       # BCC lattice constant (angstrom)
V_ATOM = A0 ** 3 / 2            # volume per atom
RIN = 0.5
SITES = {
    "bcc": [[0, 0, 0], [.5, .5, .5]],
    "fcc": [[0, 0, 0], [.5, .5, 0], [.5, 0, .5], [0, .5, .5]],
    "a15": [[0, 0, 0], [.5, .5, .5], [.25, .5, 0], [.75, .5, 0], [0, .25, .5], [0, .75, .5], [.5, 0, .25], [.5, 0, .75]],
}
# Radial, angular and body-order sizes: (L, K2, K3, K4, P3, P4).  "main" and "main23" are the models of the large
# boxes with and without the 4-body term, "small" the 2/3-body model of the 128-atom cell, "p6" the model with
# 4-body terms of degree 6, "rowN" the 2/3-body and "fourN" the 2/3/4-body models of the cost comparison's six sizes.
MODELS = {
    "small": (6, 4, 4, 0, 3, 0), "main": (8, 6, 6, 6, 4, 4), "main23": (8, 6, 6, 0, 4, 0), "p6": (8, 6, 6, 6, 4, 6),
    "row2": (8, 5, 3, 0, 2, 0), "row3": (8, 5, 5, 0, 4, 0), "row4": (8, 6, 7, 0, 6, 0), "row5": (14, 10, 9, 0, 8, 0),
    "row6": (14, 8, 12, 0, 10, 0),
    "four2": (8, 5, 3, 3, 2, 2), "four3": (8, 5, 5, 5, 4, 3), "four4": (8, 6, 7, 7, 6, 4),
}


def listed():
    return [
        # one energy and force call of a unit-cell sized system: latency and launches
        {"name": "energy_16", "kind": "energy", "model": "main", "dtype": "f64", "lattice": "bcc", "n1": 2, "n2": 2, "n3": 2, "vac": 0.0, "rcut": 5.0},
        # the benchmark's box: every output of the linear model in FP64
        {"name": "energy_15840", "kind": "energy", "model": "main", "dtype": "f64", "lattice": "bcc", "n1": 20, "n2": 20, "n3": 20, "vac": 0.01, "rcut": 5.0},
        # a training step: the differentiable energy forward, and backward to positions and coefficients
        {"name": "gradient_54000", "kind": "gradient", "model": "main", "dtype": "f32", "lattice": "bcc", "n1": 30, "n2": 30, "n3": 30, "vac": 0.0, "rcut": 5.0},
        # the largest box of the workloads, in FP32
        {"name": "energy_1024000", "kind": "energy", "model": "main", "dtype": "f32", "lattice": "bcc", "n1": 80, "n2": 80, "n3": 80, "vac": 0.0, "rcut": 5.0},
        # the same box with the network in place of the 4-body term
        {"name": "surrogate_1024000", "kind": "surrogate", "model": "main23", "dtype": "f32", "lattice": "bcc", "n1": 80, "n2": 80, "n3": 80, "vac": 0.0, "rcut": 5.0},
        # per-atom descriptors of a ragged box, as input of a fit or a network
        {"name": "descriptors_5702", "kind": "descriptors", "model": "main", "dtype": "f64", "lattice": "a15", "n1": 8, "n2": 9, "n3": 10, "vac": 0.01, "rcut": 5.0},
        # two of the larger models of the cost comparison
        {"name": "energy_row4", "kind": "energy", "model": "row4", "dtype": "f64", "lattice": "bcc", "n1": 20, "n2": 20, "n3": 20, "vac": 0.01, "rcut": 5.0},
        {"name": "energy_row6", "kind": "energy", "model": "row6", "dtype": "f64", "lattice": "bcc", "n1": 20, "n2": 20, "n3": 20, "vac": 0.01, "rcut": 5.0},
        # descriptors and their derivatives of a training set of small cells
        {"name": "batch_2000", "kind": "batch", "model": "main", "dtype": "f64", "cells": 2000, "n_max": 250, "rcut": 5.0},
        # the linear fit of that training set
        {"name": "fit_2000", "kind": "fit", "columns": 103, "cells": 2000, "rows": 751515},
        # a short trajectory from positions and velocities, its neighbour lists included
        {"name": "md_15840", "kind": "md", "model": "main", "dtype": "f64", "lattice": "bcc", "n1": 20, "n2": 20, "n3": 20, "vac": 0.01, "rcut": 5.0, "steps": 40},
        # a neighbour list and its reverse index, as before every call above
        {"name": "neighbors_15840", "kind": "neighbors", "model": "main", "dtype": "f64", "lattice": "bcc", "n1": 20, "n2": 20, "n3": 20, "vac": 0.01, "rcut": 5.0},
    ]


def _box(rng, lo, hi):
    """A lattice box of about lo to hi atoms, its edges within a factor of two of each other."""
    kind = rng.choice(sorted(SITES))
    n = math.exp(rng.uniform(math.log(lo), math.log(hi))) / len(SITES[kind])
    e = n ** (1 / 3)
    n1, n2 = (max(1, round(e * rng.uniform(0.7, 1.4))) for _ in range(2))
    n3 = max(1, int(n / (n1 * n2)))
    return {"lattice": kind, "n1": n1, "n2": n2, "n3": n3, "vac": round(rng.choice([0.0, rng.uniform(0.0, 0.03)]), 4)}


def draw(rng):
    kind = rng.choice(["energy", "energy", "energy", "gradient", "surrogate", "descriptors", "batch", "fit", "md", "neighbors"])
    if kind == "fit":
        n = math.exp(rng.uniform(math.log(20), math.log(2000)))
        return {"kind": kind, "columns": rng.choice([15, 27, 31, 37, 66, 79, 103]), "cells": int(n), "rows": 3 * int(n * rng.uniform(20, 125))}
    if kind == "batch":
        n_max = rng.choice([32, 100, 250])
        model = rng.choice(["small", "main", "main", "main23", "four2", "four3"])
        return {"kind": kind, "model": model, "dtype": "f64", "cells": int(math.exp(rng.uniform(math.log(20), math.log(2000)))), "n_max": n_max, "rcut": rng.choice([4.5, 5.0])}
    dtype = rng.choice(["f64", "f32"])
    rcut = rng.choice([4.5, 5.0, 5.0, 5.5])
    if kind == "surrogate":
        return {"kind": kind, "model": "main23", "dtype": "f32", **_box(rng, 1000, 700000), "rcut": rcut}
    if kind == "md":
        return {"kind": kind, "model": rng.choice(["small", "main", "main23", "four3"]), "dtype": "f64", **_box(rng, 500, 16000), "rcut": 5.0, "steps": rng.randint(10, 40)}
    if kind == "neighbors":
        return {"kind": kind, "model": "main", "dtype": dtype, **_box(rng, 16, 1000000), "rcut": rcut}
    model = rng.choice(["small", "main", "main", "main23", "row2", "row3", "row4", "row5", "row6", "four2", "four3", "four4", "p6"])
    most = 15000 if model in ("row5", "row6", "four4") else 100000 if model in ("row4", "p6") or dtype == "f64" else 700000
    return {"kind": kind, "model": model, "dtype": dtype, **_box(rng, 16, most), "rcut": rcut}


# ---- inputs ---------------------------------------------------------------------------------------------------------
def _np(seed, salt):
    return np.random.default_rng([int(seed), salt])


def _lattice(case, rng, sigma=0.15):
    """Displaced sites of the case's box: positions on the device (the handle's type) and the cell."""
    base = np.array(SITES[case["lattice"]], dtype=float)
    n = [case["n1"], case["n2"], case["n3"]]
    a = (len(base) * V_ATOM) ** (1 / 3)
    g = np.stack(np.meshgrid(*[np.arange(k) for k in n], indexing="ij"), -1).reshape(-1, 1, 3)
    pos = (g + base).reshape(-1, 3) * a
    drop = int(len(pos) * case["vac"])
    if drop:
        pos = pos[np.sort(rng.permutation(len(pos))[drop:])]
    pos = pos + rng.normal(0.0, sigma, pos.shape)
    return torch.tensor(pos, dtype=_type(case), device=DEV), np.diag(np.array(n) * a)


def _type(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def _training_cells(case, rng):
    """Stacked small cells of 2 to n_max atoms: BCC, FCC and A15 pieces with sites left out, volume +-10 %."""
    off, pos, cells = [0], [], []
    sizes = _np(case["cells"], 2)                               # the set's sizes and lattices belong to the case
    for _ in range(case["cells"]):
        base = np.array(SITES[sorted(SITES)[int(sizes.integers(3))]], dtype=float)
        n = int(sizes.integers(2, case["n_max"] + 1))
        a = (len(base) * V_ATOM * rng.uniform(0.9, 1.1)) ** (1 / 3)
        e = max(1, round((n / len(base)) ** (1 / 3)))
        k = [e, e, -(-n // (len(base) * e * e))]
        g = np.stack(np.meshgrid(*[np.arange(v) for v in k], indexing="ij"), -1).reshape(-1, 1, 3)
        x = ((g + base).reshape(-1, 3) * a)
        x = x[np.sort(rng.permutation(len(x))[:n])]
        pos.append(x + rng.normal(0.0, 0.1, x.shape))
        cells.append(np.diag(np.array(k) * a))
        off.append(off[-1] + n)
    return np.array(off), torch.tensor(np.concatenate(pos), device=DEV), torch.tensor(np.stack(cells), device=DEV)


def _cells_list(off, pos, cells, rcut):
    """The stacked full neighbour list (offsets, j, packed shift, r_ij) of many small orthorhombic cells."""
    n = torch.tensor(np.diff(off), device=DEV)
    first = torch.tensor(off[:-1], device=DEV)
    edge = torch.diagonal(cells, dim1=1, dim2=2)                                      # [cells, 3]
    cell_of = torch.repeat_interleave(torch.arange(len(n), device=DEV), n)
    i = torch.repeat_interleave(torch.arange(int(off[-1]), device=DEV), n[cell_of])
    start = torch.repeat_interleave(torch.cumsum(n[cell_of], 0) - n[cell_of], n[cell_of])
    j = first[cell_of[i]] + torch.arange(len(i), device=DEV) - start
    d0, e = pos[j] - pos[i], edge[cell_of[i]]
    reach = torch.ceil((rcut + d0.abs().amax(0)) / edge.amin(0)).int().tolist()
    got = []
    for s in itertools.product(*[range(-k, k + 1) for k in reach]):
        v = d0 + torch.tensor(s, dtype=torch.float64, device=DEV) * e
        r2 = (v * v).sum(1)
        at = torch.nonzero((r2 < rcut * rcut) & (r2 > 0)).squeeze(1)
        if len(at):
            sh = (s[0] & 255) | (s[1] & 255) << 8 | (s[2] & 255) << 16
            got.append((i[at], j[at], torch.full_like(at, sh), v[at]))
    i, j, sh, v = (torch.cat(x) for x in zip(*got))
    order = torch.argsort(i, stable=True)
    offsets = torch.zeros(int(off[-1]) + 1, dtype=torch.int64, device=DEV)
    offsets[1:] = torch.cumsum(torch.bincount(i, minlength=int(off[-1])), 0)
    return offsets, i[order], j[order], sh[order], v[order]


def _family(L):
    nb = L - 2
    z = np.zeros
    return (np.r_[np.arange(1.0, nb + 1), z(2)], np.r_[np.full(nb, 3.0), z(2)], np.r_[z(nb), 1.0, 2.0], np.r_[np.ones(nb), z(2)])


def _setup(case):
    L, K2, K3, K4, P3, P4 = MODELS[case["model"]]
    return pod.Setup(RIN, case["rcut"], *_family(L), K2, K3, K4, P3, P4)


def _coefficients(case, scale=1.0):
    """Coefficients of the case's model from the spread of its descriptors over a small displaced box."""
    s = _setup(case)
    cell = {"lattice": "bcc", "n1": 4, "n2": 4, "n3": 4, "vac": 0.05, "dtype": "f64"}
    D = _descriptors(s, *_lattice(cell, np.random.default_rng(8)))
    sd = D.std(0)
    m3 = s.K3 * (s.P3 + 1)
    c, rng, at = np.zeros(D.shape[1]), np.random.default_rng(5), 1
    for size, spread in ((s.K2, 1.0), (m3, 0.3), (len(sd) - 1 - s.K2 - m3, 0.1)):
        if size:
            w = sd[at:at + size].float().cpu().numpy()           # to fewer digits than the order of a sum changes
            c[at:at + size] = scale * spread * rng.normal(size=size) / (np.where(w > 0, w, 1.0) * math.sqrt(size))
            at += size
    return c, D


def prepare(case, seed):
    kind = case["kind"]
    rng = _np(seed, 1)
    if kind == "fit":
        g = torch.Generator(device=DEV).manual_seed(int(seed))
        M, rows = case["columns"], case["rows"]
        mix = torch.tensor(np.eye(M) + 0.3 * rng.normal(size=(M, M)) / math.sqrt(M), device=DEV) * torch.tensor(10.0 ** rng.uniform(-2, 2, M), device=DEV)
        G = torch.randn(case["cells"], M, generator=g, device=DEV, dtype=torch.float64) @ mix
        J = torch.randn(rows, M, generator=g, device=DEV, dtype=torch.float64) @ mix
        c = torch.tensor(rng.normal(size=M), device=DEV) / mix.abs().amax(0)
        E = G @ c + 0.05 * torch.randn(len(G), generator=g, device=DEV, dtype=torch.float64)
        F = -(J @ c) + 0.05 * torch.randn(len(J), generator=g, device=DEV, dtype=torch.float64)
        model = pod.PodModel(_setup({"model": "main", "rcut": 5.0}), "f64")
        return {"kind": kind, "model": model, "G": G, "J": J, "E": E, "F": F}
    setup = _setup(case)
    model = pod.PodModel(setup, case["dtype"], Q=_basis(setup)[:, :max(setup.K2, setup.K3, setup.K4)])
    if kind == "batch":
        off, pos, cells = _training_cells(case, rng)
        offsets, _, j, sh, _ = _cells_list(off, pos, cells, case["rcut"])
        as_int = lambda t: t.int().cpu().numpy()  # noqa: E731
        b = pod.DeviceBatch(off, pos.cpu().numpy(), cells.cpu().numpy(), as_int(offsets), as_int(j), as_int(sh))
        return {"kind": kind, "model": model, "batch": b}
    pos, cell = _lattice(case, rng)
    state = {"kind": kind, "model": model, "pos": pos, "cell": cell, "f32": case["dtype"] == "f32"}
    if kind == "neighbors":                                     # the buffers of a program that builds many lists
        cap = 64 * len(pos)
        ints = lambda n: torch.zeros(n, dtype=torch.int32, device=DEV)  # noqa: E731
        return {**state, "offsets": ints(len(pos) + 1), "nbr_j": ints(cap), "shift": ints(cap), "rev": ints(cap)}
    if kind == "md":
        c, _ = _coefficients(case, 0.02)                        # a gentle potential: forces below about 0.2 eV/A
        return {**state, "c": c, "v": _velocities(len(pos), rng), "steps": case["steps"]}
    nb = pod.DeviceNeighbors.build(model, pos, cell)
    state["nb"] = nb
    if kind == "descriptors":
        return state
    nb.build_reverse(model)
    c, D = _coefficients(case)
    state["c"] = torch.tensor(c, dtype=_type(case), device=DEV)
    if kind == "gradient":
        state["pos"].requires_grad_()
        state["c"].requires_grad_()
    if kind == "surrogate":
        net = surrogate.Network(model.M - 1, seed=3)
        net.set_standardisation(D[:, 1:])
        net.fold_output_scale(0.1, 0.0)
        state["net"] = net
    return state


def _velocities(n, rng, T=300.0):
    v = rng.normal(0.0, math.sqrt(8.617333262e-5 * T * 9.648533215665327e-3 / md.MASS_TA), (n, 3))
    return v - v.mean(0)


# ---- one pass -------------------------------------------------------------------------------------------------------
def run(s):
    kind, m = s["kind"], s["model"]
    if kind == "energy":
        o = m.energy_forces(s["pos"], s["cell"], s["nb"], s["c"], check=False)
        return {k: v.to(s["pos"].dtype) for k, v in o.items()}
    if kind == "gradient":
        s["pos"].grad = s["c"].grad = None
        E, _ = autograd.pod_energy(s["pos"], s["c"], m, s["nb"], s["cell"])
        E.backward()
        return {"E": E.detach(), "dpos": s["pos"].grad, "dc": s["c"].grad}
    if kind == "surrogate":
        o = m.energy_forces_surrogate(s["pos"], s["cell"], s["nb"], s["c"], s["net"], check=False)
        return {k: v.to(s["pos"].dtype) for k, v in o.items()}
    if kind == "descriptors":
        return m.descriptors(s["pos"], s["cell"], s["nb"], check=False)
    if kind == "batch":
        return pod.batch_assemble(m, s["batch"], check=False)
    if kind == "fit":
        M = s["G"].shape[1]
        Z = torch.empty((M + 1, M + 1), dtype=torch.float64, device=DEV)
        c, loss = torch.empty(M, dtype=torch.float64, device=DEV), torch.empty(1, dtype=torch.float64, device=DEV)
        pod.pod_fit_gram(m.h, M, len(s["G"]), s["G"], s["E"], 100.0, len(s["J"]), s["J"], s["F"], 1.0, Z)
        pod.pod_fit_solve(m.h, M, Z, 1e-12, c, loss)
        return {"Z": Z, "c": c, "loss": loss}
    if kind == "md":
        dyn = md.MD(m, s["pos"], s["v"], s["cell"], s["c"], skin=0.4)
        ep, ek = dyn.run(s["steps"], chunk=20)
        return {"x": dyn.x, "v": dyn.v, "F": dyn.F, "E_pot": ep.to(dyn.x.dtype), "E_kin": ek.to(dyn.x.dtype)}
    lst, N = (s["offsets"], s["nbr_j"], s["shift"]), len(s["pos"])
    P = pod.pod_build_neighbors(m.h, N, s["pos"], s["cell"], 0.0, *lst, capacity=s["nbr_j"].numel())
    pod.pod_neighbor_reverse(m.h, N, P, *lst, s["rev"])
    return {"offsets": s["offsets"], "nbr_j": s["nbr_j"], "shift": s["shift"], "rev": s["rev"]}


# ---- bytes and operations of one pass -------------------------------------------------------------------------------
def _counts(model):
    """Operations of a model: per pair forward, per pair backward (one weighted sum), per pair and column of the
    derivatives, per atom forward and per atom adjoint (a multiply-add is two)."""
    L, K2, K3, K4, P3, P4 = MODELS[model]
    K, PA = max(K2, K3, K4), max(P3 if K3 else 0, P4 if K4 else 0)
    Na = (PA + 1) * (PA + 2) * (PA + 3) // 6
    terms = sum(len(t) for p, t in zip(_triples(P4), _four_terms(P4)) if p[1] > 0) if K4 else 0
    M = 1 + K2 + K3 * (P3 + 1) + K4 * (len(_triples(P4)) if K4 else 0)
    return {"K": K, "M": M, "fwd": 10 * L + 30 + 2 * L * K + Na + 2 * K * Na, "bwd": 2 * L * K + 4 * K * Na + 8 * Na,
            "col": 8 * Na, "atom": K * (3 * Na + 4 * terms), "adj": K * (3 * Na + 9 * terms)}


def work(case):
    kind = case["kind"]
    if kind == "fit":
        M, rows = case["columns"] + 1, case["rows"] + case["cells"]
        return {"bytes": 8.0 * (rows * M + M * M), "flops": float(rows * M * M) + M ** 3 / 3}
    w = 8 if case["dtype"] == "f64" else 4
    near = 4 / 3 * math.pi * case["rcut"] ** 3 / V_ATOM
    if kind == "batch":
        N = case["cells"] * (case["n_max"] + 2) / 2
        k = _counts(case["model"])
        return {"bytes": 8 * N * (near + 3 + 4 * k["M"]), "flops": N * (near * (k["fwd"] + k["M"] * k["col"]) + k["atom"])}
    N = float(int(len(SITES[case["lattice"]]) * case["n1"] * case["n2"] * case["n3"] * (1 - case["vac"])))
    P = N * near
    k = _counts(case["model"])
    if kind == "neighbors":
        return {"bytes": N * (3 * w + 4) + 12 * P, "flops": 9 * P}
    if kind == "descriptors":
        return {"bytes": 8 * P + N * w * (3 + k["M"]), "flops": P * k["fwd"] + N * k["atom"]}
    flops = P * (k["fwd"] + k["bwd"]) + N * (k["atom"] + k["adj"])
    if kind == "surrogate":
        flops += N * 2 * 2 * 64 * (64 + k["M"])
    steps = 1
    if kind == "md":
        steps = case["steps"] + 1
    return {"bytes": steps * (12 * P + N * w * 7), "flops": steps * flops}


# ---- the same in 64 bits, from the defining formulas ----------------------------------------------------------------
def _snapshots(r, s):
    """f_c psi_l and its derivative for every snapshot l: two arrays [L, n]."""
    h = s.rcut - s.rin
    t = (r - s.rin) / h
    y = 1 - t ** 3
    q = y * y + 1e-6
    fc = torch.exp(1 - q ** -0.5)
    dfc = fc * y * q ** -1.5 * (-3 * t * t / h)
    d = r - s.rin
    f, df = [], []
    for a, b, g, k in zip(s.alpha, s.beta, s.gamma, s.kappa):
        if k:
            x = torch.expm1(-b * t) / math.expm1(-b)
            dx = -b * torch.exp(-b * t) / math.expm1(-b) / h
            psi = torch.sin(a * math.pi * x) / d
            dpsi = (a * math.pi * torch.cos(a * math.pi * x) * dx - psi) / d
        else:
            psi, dpsi = r ** -g, -g * r ** (-g - 1)
        f.append(fc * psi)
        df.append(dfc * psi + fc * dpsi)
    return torch.stack(f), torch.stack(df)


def _basis(s, n=2000):
    """Eigenvectors of the snapshots' correlation, by decreasing eigenvalue: the radial basis that the model is given."""
    r = s.rin + (torch.arange(n, dtype=torch.float64) + 0.5) * ((s.rcut - s.rin) / n)
    f = _snapshots(r, s)[0].numpy()
    _, V = np.linalg.eigh(f @ f.T / n)
    V = V[:, ::-1]
    return np.ascontiguousarray(V * np.sign(V[np.abs(V).argmax(0), np.arange(len(V))]))


def _pairs(pos, cell, rcut):
    """(i, j, r_ij) of every neighbour pair of an orthorhombic box, sorted by i, from bins of ghost-extended atoms."""
    edge = torch.tensor(np.diag(cell), device=DEV)
    x = pos.double()
    x = x - torch.floor(x / edge) * edge
    ids = torch.arange(len(x), device=DEV)
    gx, gi = x, ids
    for d in range(3):
        part = [(gx, gi)]
        for k in range(1, int(math.ceil(rcut / float(edge[d]))) + 1):
            for sgn in (-1, 1):
                y = gx.clone()
                y[:, d] += sgn * k * edge[d]
                keep = (y[:, d] > -rcut) & (y[:, d] < edge[d] + rcut)
                part.append((y[keep], gi[keep]))
        gx, gi = torch.cat([p[0] for p in part]), torch.cat([p[1] for p in part])
    nb = [int(math.floor(float(edge[d]) / rcut)) + 4 for d in range(3)]
    b = torch.floor(gx / rcut).long() + 1
    key = (b[:, 0] * nb[1] + b[:, 1]) * nb[2] + b[:, 2]
    order = torch.argsort(key)
    gx, gi, key = gx[order], gi[order], key[order]
    count = torch.bincount(key, minlength=nb[0] * nb[1] * nb[2])
    start = torch.cumsum(count, 0) - count
    most = int(count.max())
    slot = torch.arange(most, device=DEV)
    hb = torch.floor(x / rcut).long() + 1
    home = (hb[:, 0] * nb[1] + hb[:, 1]) * nb[2] + hb[:, 2]
    near = torch.tensor([(a * nb[1] + c) * nb[2] + e for a in (-1, 0, 1) for c in (-1, 0, 1) for e in (-1, 0, 1)], device=DEV)
    got = []
    for at in torch.split(ids, max(1, 40_000_000 // (27 * most))):
        bins = home[at][:, None] + near
        g = (start[bins][:, :, None] + slot).reshape(len(at), -1)
        live = (slot < count[bins][:, :, None]).reshape(len(at), -1)
        v = gx[g.clamp(max=len(gx) - 1)] - x[at][:, None]
        r2 = (v * v).sum(2)
        a, c = torch.nonzero(live & (r2 < rcut * rcut) & (r2 > 0), as_tuple=True)
        got.append((at[a], gi[g[a, c]], v[a, c]))
    return tuple(torch.cat(z) for z in zip(*got))


def _powers(P):
    return [(a, b, n - a - b) for n in range(P + 1) for a in range(n, -1, -1) for b in range(n - a, -1, -1)]


def _triples(P):
    return [(a, b, n - a - b) for n in range(P + 1) for a in range(n, -1, -1) for b in range(min(a, n - a), -1, -1) if 0 <= n - a - b <= b]


def _multi(e):
    return math.factorial(sum(e)) // math.prod(math.factorial(v) for v in e)


_TERMS = {}


def _four_terms(P4):
    """For each (a, b, c): {(x, y, z): weight}, the products of three basis values whose sum is the 4-body descriptor
    sum_jkl w_jk^a w_jl^b w_kl^c, each cosine power expanded by the multinomial theorem."""
    if P4 not in _TERMS:
        at = {e: n for n, e in enumerate(_powers(P4))}
        of = lambda n: [e for e in _powers(n) if sum(e) == n]  # noqa: E731
        add = lambda u, v: at[tuple(p + q for p, q in zip(u, v))]  # noqa: E731
        got = []
        for a, b, c in _triples(P4):
            t = {}
            for u, v, w in itertools.product(of(a), of(b), of(c)):
                k = tuple(sorted((add(u, v), add(u, w), add(v, w))))
                t[k] = t.get(k, 0) + _multi(u) * _multi(v) * _multi(w)
            got.append(t)
        _TERMS[P4] = got
    return _TERMS[P4]


def _monomials(u, P):
    """A [Na, n] at the unit vectors u [n, 3]."""
    p = [[torch.ones_like(u[:, d])] for d in range(3)]
    for d in range(3):
        for _ in range(P):
            p[d].append(p[d][-1] * u[:, d])
    return torch.stack([p[0][a] * p[1][b] * p[2][c] for a, b, c in _powers(P)])


def _degree(s):
    return max(s.P3 if s.K3 else 0, s.P4 if s.K4 else 0)


def _chunks(i, width):
    """Ranges of pairs of a bounded size."""
    step = max(1000, 200_000_000 // width)
    return [slice(k, min(k + step, len(i))) for k in range(0, len(i), step)]


def _density(s, i, v, N, Q):
    """Atomic basis B [K, Na, N] of the pairs (i, r_ij = v)."""
    PA, K = _degree(s), Q.shape[1]
    Na = len(_powers(PA))
    B = torch.zeros(N, K * Na, dtype=torch.float64, device=DEV)
    for c in _chunks(i, K * Na):
        r = v[c].norm(dim=1)
        R = torch.tensor(Q.T.copy(), device=DEV) @ _snapshots(r, s)[0]
        A = _monomials(v[c] / r[:, None], PA)
        B.index_add_(0, i[c], (R.T[:, :, None] * A.T[:, None, :]).reshape(len(r), -1))
    return B.T.reshape(K, Na, N).contiguous()


def _columns(s, B):
    """Descriptors [N, M] from the basis."""
    E = _powers(_degree(s))
    N = B.shape[2]
    D = [torch.ones(1, N, dtype=torch.float64, device=DEV), B[:s.K2, 0]]
    mult = torch.tensor([float(_multi(e)) for e in E], device=DEV, dtype=torch.float64)
    deg = torch.tensor([sum(e) for e in E], device=DEV)
    for m in range(s.K3):
        sq = mult[:, None] * B[m] ** 2
        D.append(torch.stack([sq[deg == n].sum(0) for n in range(s.P3 + 1)]))
    for m in range(s.K4):
        D.append(torch.stack([sum(w * B[m, x] * B[m, y] * B[m, z] for (x, y, z), w in t.items()) for t in _four_terms(s.P4)]))
    return torch.cat(D).T.contiguous()


def _jacobian(s, B, m, weights=None):
    """dD/dB of radial index m: [columns of m, Na, N], or their sum [Na, N] with the columns' weights (order: the 2-body
    column, P3 + 1 of three bodies, then the 4-body ones, as far as the model has them for m)."""
    E = _powers(_degree(s))
    b = B[m]
    rows, at = [], 0

    def put(fill):
        nonlocal at
        if weights is None:
            row = torch.zeros_like(b)
            fill(row, 1.0)
            rows.append(row)
        else:
            fill(total, weights[at])
        at += 1

    total = torch.zeros_like(b)
    if m < s.K2:
        def two(row, w):
            row[0] += w
        put(two)
    if m < s.K3:
        for n in range(s.P3 + 1):
            def three(row, w):
                for k, e in enumerate(E):
                    if sum(e) == n:
                        row[k] += 2 * w * _multi(e) * b[k]
            put(three)
    if m < s.K4:
        for t in _four_terms(s.P4):
            def four(row, w):
                for (x, y, z), q in t.items():
                    row[x] += (w * q) * b[y] * b[z]
                    row[y] += (w * q) * b[x] * b[z]
                    row[z] += (w * q) * b[x] * b[y]
            put(four)
    return total if weights is not None else torch.stack(rows) if rows else b[:0][None][:0]


def _columns_of(s, m):
    """Where the columns of radial index m stand in D, in the order of _jacobian."""
    k4 = len(_triples(s.P4)) if s.K4 else 0
    o3 = 1 + s.K2
    o4 = o3 + s.K3 * (s.P3 + 1)
    return ([1 + m] if m < s.K2 else []) + [o3 + m * (s.P3 + 1) + n for n in range(s.P3 + 1) if m < s.K3] + [o4 + m * k4 + p for p in range(k4) if m < s.K4]


def _slopes(s, v, Q):
    """R [K, n], R' [K, n], u [n, 3], A [Na, n] and r [n] of pairs."""
    r = v.norm(dim=1)
    f, df = _snapshots(r, s)
    q = torch.tensor(Q.T.copy(), device=DEV)
    u = v / r[:, None]
    return q @ f, q @ df, u, _monomials(u, _degree(s)), r


def _turn(s, A, u):
    """dA/du_d - (u . grad A) u_d = dA/du_d - deg A u_d, of the monomials as polynomials: [3, Na, n]."""
    E = _powers(_degree(s))
    at = {e: n for n, e in enumerate(E)}
    deg = torch.tensor([float(sum(e)) for e in E], device=DEV, dtype=torch.float64)[:, None]
    out = []
    for d in range(3):
        low = torch.zeros_like(A)
        for k, e in enumerate(E):
            if e[d]:
                low[k] = e[d] * A[at[tuple(v - (q == d) for q, v in enumerate(e))]]
        out.append(low - deg * A * u[:, d])
    return torch.stack(out)


def _energy(s, pos, cell, c, extra=None):
    """E_atom [N], F [N, 3], W [3, 3], G [M] of the linear model; extra(D) gives an energy per atom to add and its
    gradient [N, M] (the network's)."""
    Q = _basis(s)[:, :max(s.K2, s.K3, s.K4)]
    i, j, v = _pairs(pos, cell, s.rcut)
    N = len(pos)
    B = _density(s, i, v, N, Q)
    D = _columns(s, B)
    E = D @ c
    wt = c[None, :].expand(N, -1)
    if extra is not None:
        y, dy = extra(D)
        E, wt = E + y, wt + dy
    K, Na, _ = B.shape
    G = D.sum(0)
    adj = torch.stack([_jacobian(s, B, m, wt[:, _columns_of(s, m)].T) for m in range(K)])
    del B, D
    adj = adj.permute(2, 0, 1).contiguous()                                            # [N, K, Na]
    F, W = torch.zeros(N, 3, dtype=torch.float64, device=DEV), torch.zeros(3, 3, dtype=torch.float64, device=DEV)
    for p in _chunks(i, K * Na):
        R, dR, u, A, r = _slopes(s, v[p], Q)
        a = adj[i[p]]
        w1, w2 = (a * dR.T[:, :, None]).sum(1).T, (a * R.T[:, :, None]).sum(1).T        # [Na, n]
        g = (w1 * A).sum(0)[:, None] * u + ((w2 * _turn(s, A, u)).sum(1) / r).T
        F.index_add_(0, i[p], g)
        F.index_add_(0, j[p], -g)
        W -= v[p].T @ g
    return E, F, W, G


def _descriptors(s, pos, cell):
    Q = _basis(s)[:, :max(s.K2, s.K3, s.K4)]
    i, _, v = _pairs(pos, cell, s.rcut)
    return _columns(s, _density(s, i, v, len(pos), Q))


def _network(net, s, D):
    """Output and input gradient of the SiLU network at the standardised descriptors."""
    n, H = s, surrogate.HIDDEN
    th = net.theta.double()
    W1, b1 = th[:H * n].reshape(H, n), th[H * n:H * n + H]
    o = H * n + H
    W2, b2, w3, b3 = th[o:o + H * H].reshape(H, H), th[o + H * H:o + H * H + H], th[o + H * H + H:-1], th[-1]
    x = (D[:, 1:] - net.mu.double()) * net.inv_sigma.double()
    z1 = x @ W1.T + b1
    z2 = torch.nn.functional.silu(z1) @ W2.T + b2
    slope = lambda z: torch.sigmoid(z) * (1 + z * (1 - torch.sigmoid(z)))  # noqa: E731
    y = torch.nn.functional.silu(z2) @ w3 + b3
    dx = ((w3 * slope(z2)) @ W2 * slope(z1)) @ W1 * net.inv_sigma.double()
    return y, torch.cat([torch.zeros_like(dx[:, :1]), dx], 1)


def exact(case, seed):
    kind = case["kind"]
    rng = _np(seed, 1)
    if kind == "neighbors":
        return None
    if kind == "fit":
        s = prepare(case, seed)
        A = torch.cat([10.0 * torch.cat([s["G"], s["E"][:, None]], 1), torch.cat([-s["J"], s["F"][:, None]], 1)])
        Z = A.T @ A
        M = len(Z) - 1
        d = Z.diagonal()[:M].rsqrt()
        c = d * torch.linalg.solve(d[:, None] * Z[:M, :M] * d + 1e-12 * torch.diag(d * d), d * Z[:M, M])
        res = A[:, :M] @ c - A[:, M]
        return {"Z": Z, "c": c, "loss": (res * res).sum().reshape(1) + 1e-12 * (c * c).sum()}
    s = _setup(case)
    Q = _basis(s)[:, :max(s.K2, s.K3, s.K4)]
    if kind == "batch":
        off, pos, cells = _training_cells(case, rng)
        _, i, j, _, v = _cells_list(off, pos, cells, case["rcut"])
        N = int(off[-1])
        B = _density(s, i, v, N, Q)
        D = _columns(s, B)
        of = torch.repeat_interleave(torch.arange(len(off) - 1, device=DEV), torch.tensor(np.diff(off), device=DEV))
        G = torch.zeros(len(off) - 1, D.shape[1], dtype=torch.float64, device=DEV).index_add_(0, of, D)
        J = torch.zeros(N, 3, D.shape[1], dtype=torch.float64, device=DEV)
        for m in range(B.shape[0]):
            cols = _columns_of(s, m)
            jac = _jacobian(s, B, m).permute(2, 0, 1).contiguous()                      # [N, columns, Na]
            part = torch.zeros(N, 3 * len(cols), dtype=torch.float64, device=DEV)
            for p in _chunks(i, 2 * jac[0].numel()):
                R, dR, u, A, r = _slopes(s, v[p], Q)
                T = dR[m] * A * u.T[:, None] + (R[m] / r) * _turn(s, A, u)              # [3, Na, n]
                g = torch.matmul(jac[i[p]], T.permute(2, 1, 0).contiguous()).transpose(1, 2).reshape(len(r), -1)
                part.index_add_(0, j[p], g)
                part.index_add_(0, i[p], -g)
            J[:, :, cols] += part.reshape(N, 3, -1)
        return {"D": D, "G": G, "dGdR": J.reshape(3 * N, -1)}
    pos, cell = _lattice(case, rng)
    if kind == "descriptors":
        return _descriptors(s, pos, cell)
    if kind == "md":
        c = torch.tensor(_coefficients(case, 0.02)[0], device=DEV).to(_type(case)).double()
        x, v = pos.double(), torch.tensor(_velocities(len(pos), rng), device=DEV).to(_type(case)).double()
        f, ep, ek, acc = _energy(s, x, cell, c)[1], [], [], 9.648533215665327e-3 / md.MASS_TA
        for _ in range(case["steps"]):
            v = v + 0.5 * acc * f
            x = x + v
            e, f, _, _ = _energy(s, x, cell, c)
            v = v + 0.5 * acc * f
            ep.append(e.sum())
            ek.append(0.5 / acc * (v * v).sum())
        return {"x": x, "v": v, "F": f, "E_pot": torch.stack(ep), "E_kin": torch.stack(ek)}
    c, D0 = _coefficients(case)
    c = torch.tensor(c, device=DEV).to(_type(case)).double()
    if kind == "surrogate":
        net = surrogate.Network(len(c) - 1, seed=3)
        net.set_standardisation(D0[:, 1:])
        net.fold_output_scale(0.1, 0.0)
        E, F, W, _ = _energy(s, pos.double(), cell, c, lambda D: _network(net, len(c) - 1, D))
        return {"E": E.sum().reshape(1), "E_atom": E, "F": F, "W": W}
    E, F, W, G = _energy(s, pos.double(), cell, c)
    if kind == "gradient":
        return {"E": E.sum(), "dpos": -F, "dc": G}
    return {"E": E.sum().reshape(1), "E_atom": E, "F": F, "W": W, "G": G}

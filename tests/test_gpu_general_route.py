"""The per-atom and pair kernels against the oracle.  Systems of the size of the
parity and edge tests run in one workgroup per atom, so here each system is
stacked to copies that are together above that route's largest size, and every
copy is compared with the oracle's values of the one system.  Same inputs and
same tolerances as those tests (FP64 1e-10 of the largest entry; FP32 2e-5
energies, 1e-4 forces, virial and G, 1e-3 a descriptor column)."""
import numpy as np
import pytest
import torch

from gpu_common import Case, colerr, positions_for, relerr, reverse_index, say
from oracle import pod_oracle as po
from paper_2212_14446_amd import pod, workloads as wl
from test_gpu_edges import S, _raises, _small
from test_gpu_parity import SWEEP, box49  # noqa: F401  (box49: the 49-atom box of the sweep)

pytestmark = pytest.mark.gpu

LARGEST = 1024      # atoms up to which the small route may take a call


def _stack(pos, nl, copies):
    N, P = len(pos), nl.n_pairs
    big = np.arange(copies)[:, None]
    off = np.concatenate([(nl.offsets[:-1].astype(np.int64) + big * P).ravel(), [copies * P]])
    return np.tile(pos, (copies, 1)), pod.DeviceNeighbors(off, (nl.nbr_j.astype(np.int64) + big * N).ravel(),
                                                          np.tile(nl.shift, copies))


def _errors(case, dtype):
    """Worst error over the copies of every output, on both force paths."""
    pos = positions_for(dtype, case.pos)
    c = case.c if dtype == "f64" else case.c.astype(np.float32).astype(np.float64)
    case = Case(pos, case.cell, case.nl, case.setup, c, case.name)
    N = len(pos)
    copies = LARGEST // N + 1
    big, nb = _stack(pos, case.nl, copies)
    m = case.model(dtype)
    D_ref, o_ref = case.oracle_descriptors(), case.oracle_ef()
    cpu = lambda t: t.double().cpu().numpy()  # noqa: E731
    D = cpu(m.descriptors(big, case.cell, nb)).reshape(copies, N, -1)
    errs = {"D": max(colerr(d, D_ref) for d in D)}
    for path in ("atomic", "gather"):
        if path == "gather":
            rev = nb.build_reverse(m).cpu().numpy().reshape(copies, -1)
            assert np.array_equal(rev, reverse_index(case.nl) + np.arange(copies)[:, None] * case.nl.n_pairs)
        o = {k: cpu(v) for k, v in m.energy_forces(big, case.cell, nb, case.c).items()}
        for k in ("E_atom", "F"):
            errs[f"{k} {path}"] = max(relerr(x, o_ref[k]) for x in o[k].reshape(copies, *np.shape(o_ref[k])))
        errs[f"E {path}"] = abs(o["E"][0] / copies - o_ref["E"]) / abs(o_ref["E"])
        for k in ("W", "G"):
            errs[f"{k} {path}"] = relerr(o[k] / copies, o_ref[k])
    # energies alone: an instance of their own
    o = {k: cpu(v) for k, v in m.energy_forces(big, case.cell, nb, case.c, forces=False, virial=False).items()
         if v is not None}
    errs["E_atom alone"] = max(relerr(x, o_ref["E_atom"]) for x in o["E_atom"].reshape(copies, N))
    errs["E alone"] = abs(o["E"][0] / copies - o_ref["E"]) / abs(o_ref["E"])
    errs["G alone"] = relerr(o["G"] / copies, o_ref["G"])
    say(f"[gpu] general route {case.name} {dtype} N={copies * N}: " + " ".join(f"{k}={v:.1e}" for k, v in errs.items()))
    return errs


def _hold(errs, dtype):
    for k, v in errs.items():
        tol = 1e-10 if dtype == "f64" else {"E": 2e-5, "D": 1e-3}.get(k.split("_")[0].split()[0], 1e-4)
        assert v < tol, (k, v)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("L,K2,K3,K4,P3,P4", SWEEP)
def test_sweep(box49, L, K2, K3, K4, P3, P4, dtype):  # noqa: F811
    pos, cell = box49
    s = wl.PodSetup(0.5, 5.0, L, K2, K3, K4, P3, P4)
    c = wl.coefficients(s.M, seed=(100 if dtype == "f64" else 200) + L + K2 + 3 * K3 + 5 * K4 + 7 * P3 + 11 * P4)
    case = Case(pos, cell, wl.neighbor_list(pos, cell, s.rcut), s, c, f"L{L}_K{K2}{K3}{K4}_P{P3}{P4}")
    _hold(_errors(case, dtype), dtype)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_general_snapshot_family(box49, dtype):  # noqa: F811
    pos, cell = box49
    s = pod.Setup(0.4, 4.8,
                  np.array([1.0, 2.0, 1.5, 4.0, 3.0, 2.0, 0.0, 1.0]),
                  np.array([3.0, 3.0, 3.0, 3.0, 3.0, 1.0, 0.0, 0.0]),
                  np.array([0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 2.5, 1.0]),
                  np.array([1.0, 1.0, 1.0, 0.6, 1.0, 1.0, 0.0, 1.0]),
                  5, 4, 3, 3, 3)
    M = po.num_descriptors(po.PodParams(s.rin, s.rcut, s.alpha, s.beta, s.gamma, s.kappa,
                                        s.K2, s.K3, s.K4, s.P3, s.P4))[0]
    case = Case(pos, cell, wl.neighbor_list(pos, cell, s.rcut), s, wl.coefficients(M, seed=5), "general_snapshots")
    _hold(_errors(case, dtype), dtype)


@pytest.mark.parametrize("n", [1, 2])
def test_self_images(n):
    pos, cell = wl.bcc(n)
    pos = wl.displace(pos, 0.1, 5)
    case = Case(pos, cell, wl.neighbor_list(pos, cell, S.rcut), S, wl.coefficients(S.M, 4), f"bcc{n}_self_images")
    _hold(_errors(case, "f64"), "f64")


def test_open_system_with_isolated_atoms():
    pos, _ = wl.lattice("bcc", 2, 2, 1, 3.31)
    pos = np.vstack([pos + np.random.default_rng(3).normal(0, 0.1, pos.shape), [[40.0, 40.0, 40.0], [-30.0, 0.0, 0.0]]])
    case = Case(pos, None, wl.neighbor_list(pos, None, S.rcut), S, wl.coefficients(S.M, 9), "open_isolated")
    _hold(_errors(case, "f64"), "f64")


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_skin_list(dtype):
    """A list with a skin gives the exact list's results (1e-12, 1e-5 as on the
    small route)."""
    pos, cell = _small()
    m = pod.PodModel(pod.setup_from_workload(S), dtype)
    c = wl.coefficients(S.M, 3)
    copies = LARGEST // len(pos) + 1
    out = []
    for skin in (0.0, 0.6):
        big, nb = _stack(pos, wl.neighbor_list(pos, cell, S.rcut + skin), copies)
        o = {"D": m.descriptors(big, cell, nb), **m.energy_forces(big, cell, nb, c)}
        nb.build_reverse(m)
        o["F gather"] = m.energy_forces(big, cell, nb, c)["F"]
        out.append({k: v.double().cpu().numpy() for k, v in o.items()})
    say(f"[gpu] general route, skin list {dtype}")
    tol = 1e-12 if dtype == "f64" else 1e-5
    for k in out[0]:
        assert (colerr if k == "D" else relerr)(out[1][k], out[0][k]) < tol, k


def test_data_errors():
    """Malformed lists, a pair inside rin and a non-finite position in one copy."""
    pos, cell = _small()
    nl = wl.neighbor_list(pos, cell, S.rcut)
    m = pod.PodModel(pod.setup_from_workload(S), "f64")
    c = np.ones(m.M)
    copies = LARGEST // len(pos) + 1
    say("[gpu] general route, data errors")

    def both(code, x, cl, off=None, j=None):
        big, nb = _stack(pos, nl, copies)
        if x is not None:
            big[len(pos) * (copies - 2):len(pos) * (copies - 1)] = x
        if off is not None or j is not None:
            o, jj = nb.offsets.cpu().numpy().copy(), nb.nbr_j.cpu().numpy().copy()
            if off is not None:
                o[off[0]] = off[1](o)
            if j is not None:
                jj[j[0]] = j[1]
            nb = pod.DeviceNeighbors(o, jj, nb.shift.cpu().numpy())
        _raises(code, lambda: m.descriptors(big, cl, nb))
        _raises(code, lambda: m.energy_forces(big, cl, nb, c))
        _raises(code, lambda: m.energy_forces(big, cl, nb, c, forces=False, virial=False))
        m.check()

    near = pos.copy()
    k = int(nl.nbr_j[0])
    near[0] = pos[k] + nl.shift3[0] @ cell - np.array([0.3, 0.0, 0.0])
    both("POD_ERANGE", near, cell)
    nan = pos.copy()
    nan[3, 1] = np.nan
    both("POD_ENONFINITE", nan, cell)
    both("POD_ENEIGH", None, cell, j=(5, copies * len(pos) + 3))
    both("POD_ENEIGH", None, cell, off=(900, lambda o: o[902] + 1))
    both("POD_ENEIGH", None, None)              # an open system with image shifts


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("copies", [10, 11, 20, 21])
@pytest.mark.parametrize("K2, K3, K4, P3, P4", [(4, 4, 4, 3, 3), (6, 6, 6, 4, 4)])
def test_launch_shapes_of_the_small_route(box49, K2, K3, K4, P3, P4, copies, dtype):  # noqa: F811
    """490 and 539 atoms (256 and 128 threads per atom) and 980 and 1,029 (one
    workgroup per atom, per-atom kernel): every copy against the oracle."""
    pos, cell = box49
    s = wl.PodSetup(0.5, 5.0, 8, K2, K3, K4, P3, P4)
    x = positions_for(dtype, pos)
    c = wl.coefficients(s.M, 7)
    c = c if dtype == "f64" else c.astype(np.float32).astype(np.float64)
    case = Case(x, cell, wl.neighbor_list(x, cell, s.rcut), s, c)
    m = case.model(dtype)
    o_ref, D_ref = case.oracle_ef(), case.oracle_descriptors()
    big, nb = _stack(x, case.nl, copies)
    say(f"[gpu] launch shape N={len(big)} {dtype} K={K2}")
    D = m.descriptors(big, cell, nb).double().cpu().numpy().reshape(copies, len(x), -1)
    f64 = dtype == "f64"
    assert max(colerr(d, D_ref) for d in D) < (1e-10 if f64 else 1e-3)
    for gather in (False, True):
        if gather:
            nb.build_reverse(m)
        o = {k: v.double().cpu().numpy() for k, v in m.energy_forces(big, cell, nb, c).items()}
        assert max(relerr(f, o_ref["F"]) for f in o["F"].reshape(copies, -1, 3)) < (1e-10 if f64 else 1e-4)
        assert max(relerr(e, o_ref["E_atom"]) for e in o["E_atom"].reshape(copies, -1)) < (1e-10 if f64 else 2e-5)
        for k in ("W", "G"):
            assert relerr(o[k] / copies, o_ref[k]) < (1e-10 if f64 else 1e-4), k

"""One workgroup per atom (few atoms) against the per-atom and pair kernels
(many): the same system once by itself and once as copies stacked into one
call that is too large for the small path.  Every copy must reproduce the
single system.  The single system is pinned to the oracle by the parity tests;
this test covers the models, list lengths (a chunk of staged pairs, one more,
several chunks, none) and force paths at which the two routes split.

Tolerance: both routes are FP64 (FP32) evaluations of the same sums in other
orders over at most a few hundred terms; 1e-11 (2e-5 energies, 1e-4 forces, the
stated FP32 bounds) of the largest entry."""
import numpy as np
import pytest
import torch

from gpu_common import say
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu


def _system(rcut, n, seed):
    pos, cell = wl.lattice("bcc", n, n, n, 3.31)
    pos = wl.displace(pos, 0.12, seed)
    return pos, cell, wl.neighbor_list(pos, cell, rcut)


def _stack(pos, nl, copies):
    N, P = len(pos), nl.n_pairs
    off = np.concatenate([nl.offsets[:-1].astype(np.int64) + c * P for c in range(copies)] + [[copies * P]])
    j = (nl.nbr_j[None].astype(np.int64) + np.arange(copies)[:, None] * N).ravel()
    return np.tile(pos, (copies, 1)), pod.DeviceNeighbors(off, j, np.tile(nl.shift, copies))


def _rel(x, ref):
    return float((x.double() - ref.double()).abs().max() / ref.double().abs().max().clamp(min=1e-30))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("K2, K3, K4, P3, P4, rcut", [
    (3, 0, 0, 0, 0, 5.0),        # 2-body only
    (1, 1, 1, 1, 1, 5.0),
    (4, 4, 0, 3, 0, 5.0),
    (5, 3, 3, 2, 2, 6.9),        # about 58 to 65 pairs: around one chunk of 64
    (6, 6, 6, 4, 4, 7.6),        # about 88 to 113 pairs: two chunks
    (2, 8, 5, 4, 3, 5.0),
    (3, 2, 4, 3, 5, 5.0),        # degree 5 and 6: chunks of 32
    (6, 7, 2, 6, 4, 5.4),
    (2, 2, 3, 2, 6, 3.2),        # 8 pairs
])
def test_small_against_general(K2, K3, K4, P3, P4, rcut, dtype):
    s = wl.PodSetup(0.5, rcut, 8, K2, K3, K4, P3, P4)
    m = pod.PodModel(pod.setup_from_workload(s), dtype)
    pos, cell, nl = _system(rcut, 3, 5)
    N = len(pos)
    say(f"[gpu] small vs general K=({K2},{K3},{K4}) P=({P3},{P4}) rcut={rcut} {dtype} pairs/atom="
        f"{np.diff(nl.offsets).min()}..{np.diff(nl.offsets).max()}")
    c = wl.coefficients(s.M, 3)
    tol_e, tol_f = (1e-11, 1e-11) if dtype == "f64" else (2e-5, 1e-4)
    one = pod.DeviceNeighbors.from_list(nl)
    for copies in (6, 20, 24):      # one route, the other, and the next launch shape
        big, nb = _stack(pos, nl, copies)
        D1, D = m.descriptors(pos, cell, one), m.descriptors(big, cell, nb)
        for k in range(copies):
            assert _rel(D[k * N:(k + 1) * N], D1) < tol_f
        for gather in (True, False):
            for x in (one, nb):
                x.rev = None
                if gather:
                    x.build_reverse(m)
            a, b = m.energy_forces(pos, cell, one, c), m.energy_forces(big, cell, nb, c)
            assert _rel(b["E"] / copies, a["E"]) < tol_e
            assert _rel(b["G"] / copies, a["G"]) < tol_e
            assert _rel(b["W"] / copies, a["W"]) < tol_f
            for k in range(copies):
                assert _rel(b["E_atom"][k * N:(k + 1) * N], a["E_atom"]) < tol_e
                assert _rel(b["F"][k * N:(k + 1) * N], a["F"]) < tol_f


@pytest.mark.parametrize("N", [1, 511, 512, 513, 1023, 1024, 1025])
def test_route_edges(N):
    """Open clusters of N atoms (the first alone) on both sides of every switch,
    against two half-size calls that stay on the small path."""
    s = wl.PodSetup(0.5, 4.0, 6, 3, 3, 2, 3, 2)
    m = pod.PodModel(pod.setup_from_workload(s), "f64")
    pos, _ = wl.lattice("bcc", 9, 9, 9, 3.31)
    pos = wl.displace(pos[:N], 0.1, 2)
    pos[0] -= 100.0
    say(f"[gpu] small route N={N}")
    nl = wl.neighbor_list(pos, None, s.rcut)
    c = wl.coefficients(s.M, 4)
    nb = pod.DeviceNeighbors.from_list(nl)
    if nl.n_pairs:
        nb.build_reverse(m)
    o = m.energy_forces(pos, None, nb, c)
    D = m.descriptors(pos, None, nb)
    assert float((D @ torch.as_tensor(c, device="cuda") - o["E_atom"]).abs().max()) < 1e-11 * float(o["E_atom"].abs().max())
    assert abs(float(o["E_atom"].sum() - o["E"][0])) < 1e-11 * float(o["E_atom"].abs().sum())
    assert float((D.sum(0) - o["G"]).abs().max()) < 1e-11 * float(o["G"].abs().max())
    assert float(o["F"].sum(0).abs().max()) <= 1e-11 * max(float(o["F"].abs().sum()), 1e-30)
    quarter = min(N, 300)
    near = pod.DeviceNeighbors(nl.offsets[:quarter + 1], nl.nbr_j[:nl.offsets[quarter]], nl.shift[:nl.offsets[quarter]])
    # rows of the first atoms from a call over those atoms only, as long as their neighbours are among them
    inside = [i for i in range(quarter) if all(j < quarter for j in nl.nbr_j[nl.offsets[i]:nl.offsets[i + 1]])]
    Dq = m.descriptors(pos[:quarter], None, near, check=False)
    try:
        m.check()
    except pod.PodError:
        pass                      # neighbours outside the shortened call are reported and skipped
    assert _rel(Dq[inside], D[inside]) < 1e-11

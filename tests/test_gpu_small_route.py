"""Both sides of the rule that sends a small system to one workgroup per atom:
lists from none to several rounds of the per-atom kernel, each call alone and as
copies in a system above every threshold.  Descriptors, energy alone and forces
may take different kernels; all must agree.  FP64, sums of at most a few hundred
terms in another order: 1e-11 of the largest entry."""
import numpy as np
import pytest
import torch

from gpu_common import say
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu


def _near(x, ref):
    assert float((x - ref).abs().max()) <= 1e-11 * max(float(ref.abs().max()), 1e-30)


@pytest.mark.parametrize("K2, K3, K4, P3, P4", [(4, 4, 0, 3, 0), (8, 8, 8, 4, 4), (3, 3, 3, 2, 5), (6, 7, 0, 6, 0)])
@pytest.mark.parametrize("box", [(3, 3, 3), (8, 8, 5)])
def test_short_lists(K2, K3, K4, P3, P4, box):
    s = wl.PodSetup(0.5, 5.2, 10, K2, K3, K4, P3, P4)
    m = pod.PodModel(pod.setup_from_workload(s), "f64")
    K = max(K2, K3, K4)
    c = wl.coefficients(s.M, 3)
    pos, cell = wl.lattice("bcc", *box, 3.31)
    pos = wl.displace(pos, 0.1, 5)
    nl = wl.neighbor_list(pos, cell, s.rcut)
    N, copies = len(pos), 1100 // len(pos) + 1
    place = np.arange(nl.n_pairs) - np.repeat(nl.offsets[:-1], np.diff(nl.offsets))
    for pairs in (0, 1, K - 1, K, 2 * K - 1, 2 * K, 5 * K // 2 + 1, 3 * K):
        keep = place < pairs              # the first entries of every row
        cnt = np.minimum(np.diff(nl.offsets), pairs)
        off = np.concatenate([[0], np.cumsum(cnt)]).astype(np.int64)
        j, sh, P = nl.nbr_j[keep], nl.shift[keep], int(off[-1])
        big = np.arange(copies)[:, None]
        one = pod.DeviceNeighbors(off, j, sh)
        many = pod.DeviceNeighbors(np.concatenate([(off[:-1] + big * P).ravel(), [copies * P]]), (j + big * N).ravel(),
                                   np.tile(sh, copies))
        say(f"[gpu] small route K={K} four={K4 > 0} N={N} P={P}")
        D = m.descriptors(pos, cell, one)
        E = m.energy_forces(pos, cell, one, c, forces=False, virial=False)
        F = m.energy_forces(pos, cell, one, c)
        tile = np.tile(pos, (copies, 1))
        _near(m.descriptors(tile, cell, many).view(copies, N, -1), D)
        B = m.energy_forces(tile, cell, many, c)
        for k in ("E_atom", "F"):
            _near(B[k].view(copies, *F[k].shape), F[k])
        for k in ("E", "W", "G"):
            _near(B[k] / copies, F[k])
        for k in ("E", "E_atom", "G"):
            _near(E[k], F[k])
        _near(D @ torch.as_tensor(c, device="cuda"), F["E_atom"])

"""More atoms than one launch of the neighbour search takes (2^27, 16 lanes
each): a sparse lattice with a few close pairs at the ends and at the seam."""
import numpy as np
import pytest
import torch

from gpu_common import say
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu


def test_search_in_slices():
    m = pod.PodModel(pod.setup_from_workload(wl.SETUP_CFG1), "f32")
    n, a = (512, 512, 515), 3.0
    N, seam = n[0] * n[1] * n[2], 2 ** 27
    assert seam < N
    say(f"[gpu] neighbour search of {N} atoms")
    pos = torch.empty((N, 3), dtype=torch.float32, device="cuda")
    k = torch.arange(N, device="cuda")
    for d, q in enumerate((k % n[0], k // n[0] % n[1], k // (n[0] * n[1]))):
        pos[:, d] = q.float() * a
    del k, q
    for i in (0, seam, N - 2):                # neighbours in a row of the lattice, moved together
        pos[i, 0] += 1.25
        pos[i + 1, 0] = pos[i, 0] + 0.5
    want = {0: 1, 1: 0, seam: seam + 1, seam + 1: seam, N - 2: N - 1, N - 1: N - 2}
    cell = np.diag([n[0] * a, n[1] * a, n[2] * a])
    off = torch.empty(N + 1, dtype=torch.int32, device="cuda")
    j = torch.full((8,), -1, dtype=torch.int32, device="cuda")
    sh = torch.full((8,), -1, dtype=torch.int32, device="cuda")
    P = pod.pod_build_neighbors(m.h, N, pos, cell, 1.0, off, j, sh, 8)
    pod.pod_check(m.h)
    assert P == len(want)
    got = torch.nonzero(off[1:] - off[:-1]).squeeze(1).cpu().tolist()
    assert got == sorted(want)
    assert j[:P].cpu().tolist() == [want[i] for i in got] and not sh[:P].any()
    assert int(off[-1]) == P

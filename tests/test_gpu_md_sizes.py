"""Kicks inside the force gather behind the per-atom and pair kernels, beyond
4,096 atoms (more partial sums than the separate kernels have), past one ring
of 64 steps, and on both sides of the 32,768-atom switch, against the separate
kernels (no reverse index).  The two force sums differ in order only, so
trajectories agree as on small systems: 1e-11 in FP64, 2e-5 in FP32."""
import numpy as np
import pytest
import torch

from gpu_common import say
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("N, box, nsteps", [(1025, (9, 9, 9), 5), (4097, (13, 13, 13), 66), (5487, (14, 14, 14), 3),
                                            (32768, (26, 26, 26), 2), (32769, (26, 26, 26), 2)])
def test_step_with_and_without_reverse_index(N, box, nsteps, dtype):
    say(f"[gpu] md N={N} steps={nsteps} {dtype}")
    s = wl.PodSetup(0.5, 5.0, 8, 4, 4, 4, 3, 3)
    m = pod.PodModel(pod.setup_from_workload(s), dtype)
    rng = np.random.default_rng(N)
    pos, cell = wl.lattice("bcc", *box, 3.3)
    pos = wl.displace(pos, 0.05, 3)[np.sort(rng.permutation(len(pos))[:N])]
    assert len(pos) == N
    x0 = torch.as_tensor(pos, dtype=m.torch_dtype, device="cuda")
    v0 = torch.as_tensor(rng.normal(scale=1e-3, size=(N, 3)), dtype=m.torch_dtype, device="cuda")
    c = torch.as_tensor(rng.normal(scale=1e-3, size=m.M), dtype=m.torch_dtype, device="cuda")
    nb = pod.DeviceNeighbors.build(m, x0, cell, rlist=5.4)
    nb.build_reverse(m)
    F0 = m.energy_forces(x0, cell, nb, c)["F"]
    res = []
    for rev in (nb.rev, None):
        x, v, F = x0.clone(), v0.clone(), F0.clone()
        ep, ek = (torch.empty(nsteps, dtype=torch.float64, device="cuda") for _ in range(2))
        disp = torch.empty(1, dtype=torch.float64, device="cuda")
        pod.pod_md_verlet(m.h, N, nb.P, x, v, F, cell, nb.offsets, nb.nbr_j, nb.shift, rev, c, 180.9, 1.0, nsteps,
                          ep, ek, x0, disp)
        m.check()
        res.append([t.double().cpu().numpy() for t in (x, v, F, ep, ek, disp)])
    tol = 1e-11 if dtype == "f64" else 2e-5
    for a, b in zip(*res):
        assert np.abs(a - b).max() <= tol * max(np.abs(b).max(), 1e-30)
    x = res[0][0]
    d = np.linalg.norm(x - x0.double().cpu().numpy(), axis=1).max()
    assert res[0][5][0] >= d * (1 - 1e-12)

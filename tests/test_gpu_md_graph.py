"""A molecular-dynamics step captured in a graph stays valid when the same
handle serves a larger system in between: its scratch must not move."""
import numpy as np
import pytest
import torch

from gpu_common import say
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu


def _box(m, n, seed):
    pos, cell = wl.bcc(n)
    rng = np.random.default_rng(seed)
    x = torch.as_tensor(wl.displace(pos, 0.05, seed), dtype=torch.float64, device="cuda")
    v = torch.as_tensor(rng.normal(scale=1e-3, size=x.shape), device="cuda")
    nb = pod.DeviceNeighbors.build(m, x, cell, rlist=5.4)
    nb.build_reverse(m)
    return x, v, cell, nb


def test_captured_step_survives_a_larger_system():
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        _run(st)


def _run(st):
    s = wl.PodSetup(0.5, 5.0, 8, 4, 4, 4, 3, 3)
    m = pod.PodModel(pod.setup_from_workload(s), "f64")
    c = torch.as_tensor(1e-3 * wl.coefficients(s.M, 3), device="cuda")
    (x0, v0, cell, nb), (bx0, bv0, bcell, bnb) = _box(m, 4, 1), _box(m, 15, 2)   # 128 and 6,750 atoms: 16 and 844 partial sums
    say("[gpu] md step in a graph, larger system in between")
    bF0 = m.energy_forces(bx0, bcell, bnb, c)["F"]       # the energy path's scratch has its final size from here on
    F0 = m.energy_forces(x0, cell, nb, c)["F"]
    x, v, F = x0.clone(), v0.clone(), F0.clone()
    ek = torch.zeros(2, dtype=torch.float64, device="cuda")
    disp = torch.zeros(1, dtype=torch.float64, device="cuda")

    def step():
        pod.pod_md_verlet(m.h, nb.N, nb.P, x, v, F, cell, nb.offsets, nb.nbr_j, nb.shift, nb.rev, c, 180.9, 1.0, 2,
                          None, ek, x0, disp)

    step()
    m.check()
    ref = [t.clone() for t in (x, v, F, ek, disp)]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        step()
    for _ in range(3):
        bx, bv, bF = bx0.clone(), bv0.clone(), bF0.clone()
        pod.pod_md_verlet(m.h, bnb.N, bnb.P, bx, bv, bF, bcell, bnb.offsets, bnb.nbr_j, bnb.shift, bnb.rev, c, 180.9,
                          1.0, 2)
        m.check()
        x.copy_(x0), v.copy_(v0), F.copy_(F0)
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip((x, v, F, ek, disp), ref):
            assert torch.equal(a, b)
    m.check()

"""The virial's lever arm is the pair vector itself, on every route of the
energy path.  One listed pair (0 -> 1) of two atoms, the rest alone: the forces
are +g and -g with g = dE_0/dr_01 in the handle's type, and the virial is
-r_01 (x) g, one product of two numbers of that type each, exact in double for
FP32 and rounded once for FP64."""
import numpy as np
import pytest
import torch

from gpu_common import say
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("N", [2, 300, 700, 1100])
@pytest.mark.parametrize("K2, K3, K4, P3, P4", [(4, 4, 4, 3, 3), (3, 3, 2, 5, 2)])
def test_lever_arm(K2, K3, K4, P3, P4, N, dtype):
    s = wl.PodSetup(0.5, 5.0, 8, K2, K3, K4, P3, P4)
    m = pod.PodModel(pod.setup_from_workload(s), dtype)
    say(f"[gpu] virial of one pair N={N} {dtype} P3={P3}")
    rng = np.random.default_rng(N)
    c = torch.as_tensor(wl.coefficients(s.M, 3), dtype=m.torch_dtype, device="cuda")
    for _ in range(8):
        pos = np.zeros((N, 3))
        v = rng.normal(size=3)
        pos[1] = v / np.linalg.norm(v) * rng.uniform(1.5, 4.5)
        x = torch.as_tensor(pos, dtype=m.torch_dtype, device="cuda")
        off = np.ones(N + 1, np.int32)
        off[0] = 0
        nb = pod.DeviceNeighbors(off, np.ones(1, np.int32), np.zeros(1, np.int32))
        o = m.energy_forces(x, None, nb, c)
        g = o["F"][0].double().cpu().numpy()
        assert np.array_equal(o["F"][1].double().cpu().numpy(), -g) and np.abs(g).max() > 0
        W = -np.outer(x[1].double().cpu().numpy(), g)
        assert np.abs(o["W"].cpu().numpy() - W).max() <= 2.0 ** -52 * np.abs(W).max()

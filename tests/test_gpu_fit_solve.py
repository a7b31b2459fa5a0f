"""pod_fit_solve reads the matrix Z[:M, :M], the right-hand side Z[:M, M] and
the corner Z[M, M], as its header says: the last row left of the corner may
hold anything."""
import numpy as np
import pytest
import torch

from gpu_common import say
from oracle import fit_oracle as fo
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 2, 8, 9, 16, 17, 64, 103, 128])
def test_last_row_is_not_read(M):
    """A random problem of condition below 1e3, whose normal equations agree
    with the oracle's orthogonal solve to 1e3 x 128 x 2^-52 = 3e-11 at worst."""
    say(f"[gpu] fit solve, last row of Z not filled, M={M}")
    m = pod.PodModel(pod.setup_from_workload(wl.SETUP_CFG1), "f64")
    rng = np.random.default_rng(40 + M)
    A = rng.normal(size=(20 * M + 30, M))
    b = A @ rng.normal(size=M) + 0.1 * rng.normal(size=len(A))
    Z = fo.gram(A, b)
    Z[M, :M] = np.nan
    c = torch.empty(M, dtype=torch.float64, device="cuda")
    loss = torch.empty(1, dtype=torch.float64, device="cuda")
    for out in (loss, None):
        c.fill_(0.0)
        pod.pod_fit_solve(m.h, M, torch.as_tensor(Z, device="cuda").contiguous(), 1e-3, c, out)
        pod.pod_check(m.h)
        ref = fo.ridge_solve(A, b, 1e-3)
        assert np.abs(c.cpu().numpy() - ref).max() <= 1e-10 * np.abs(ref).max()
    assert abs(loss.item() - fo.objective(A, b, ref, 1e-3)) <= 1e-9 * float(b @ b)

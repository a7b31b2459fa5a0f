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


@pytest.mark.parametrize("M", [3, 4, 5, 6, 7, 8, 9])
def test_small_sizes_and_singular(M):
    """The one-wavefront solve (M <= 8) and the first size beyond it; a matrix
    that is not positive definite is reported, c = 0 and the loss NaN.  The
    tolerance is the one derived above."""
    say(f"[gpu] fit solve small M={M}")
    m = pod.PodModel(pod.setup_from_workload(wl.SETUP_CFG1), "f64")
    rng = np.random.default_rng(M)
    A = rng.normal(size=(20 * M, M)) * 10.0 ** rng.uniform(-3, 3, M)
    b = rng.normal(size=len(A))
    c = torch.empty(M, dtype=torch.float64, device="cuda")
    loss = torch.empty(1, dtype=torch.float64, device="cuda")
    Z = torch.as_tensor(fo.gram(A, b), device="cuda").contiguous()
    pod.pod_fit_solve(m.h, M, Z, 0.0, c, loss)
    pod.pod_check(m.h)
    ref = fo.ridge_solve(A, b, 0.0)
    scale = np.linalg.norm(A, axis=0)
    assert np.abs((c.cpu().numpy() - ref) * scale).max() <= 1e-10 * np.abs(ref * scale).max()
    assert abs(loss.item() - fo.objective(A, b, ref, 0.0)) <= 1e-9 * float(b @ b)
    for bad in ("diagonal", "pivot", "nan"):
        Y = Z.clone()
        if bad == "diagonal":
            Y[M - 1, M - 1] = -1.0
        elif bad == "pivot":                      # two columns the same but for a sign in the corner
            Y[:, 1] = Y[:, 0]
            Y[1, :] = Y[0, :]
            Y[1, 1] = 0.5 * Y[0, 0]
        else:
            Y[M - 1, 0] = float("nan")
        with pytest.raises(pod.PodError) as e:
            pod.pod_fit_solve(m.h, M, Y, 0.0, c, loss)
            pod.pod_check(m.h)
        assert pod.ERRORS[e.value.code] == "POD_ESINGULAR", bad
        assert not c.any() and torch.isnan(loss).all()

"""Monomials of the wide-degree kernel carry no error that all pairs share.  For
an atom with one neighbour the degree sums are D3_ka = R_k^2 |u|^(2a) = D2_k^2
(eq. (26a), a unit vector), so the mean of D3_ka / D2_k^2 - 1 over many random
directions keeps only what does not average out.

Tolerance in FP32: a dimer's ratio scatters by 9e-7 at degree 10 (u is rounded
to 2^-24 per component, its tenth powers ten times that), the mean of 4,096 by
9e-7 / 64 = 1.4e-8; four times that and the 2e-8 that plain FP32 powers and sums
leave: 8e-8.  In FP64 the same figures times 2^-29: 1.5e-16."""
import numpy as np
import pytest
import torch

from gpu_common import say
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype, tol", [("f32", 8e-8), ("f64", 1.5e-16)])
@pytest.mark.parametrize("K, P3", [(3, 7), (2, 10)])
def test_no_common_error(K, P3, dtype, tol):
    s = wl.PodSetup(0.5, 5.0, 8, K, K, 0, P3, 0)
    m = pod.PodModel(pod.setup_from_workload(s), dtype)
    n = 4096
    rng = np.random.default_rng(1)
    v = rng.normal(size=(n, 3))
    v *= (rng.uniform(1.5, 3.0, n) / np.linalg.norm(v, axis=1))[:, None]
    pos = np.zeros((2 * n, 3))
    pos[1::2] = v
    x = torch.as_tensor(pos, dtype=m.torch_dtype, device="cuda")
    j = np.arange(2 * n).reshape(n, 2)[:, ::-1].ravel()
    nb = pod.DeviceNeighbors(np.arange(2 * n + 1), j, np.zeros(2 * n, np.int32))
    D = m.descriptors(x, None, nb)[::2].cpu().numpy().astype(np.longdouble)
    D2, D3 = D[:, 1:1 + K], D[:, 1 + K:].reshape(n, K, P3 + 1)
    far = np.abs(D2[:, 0]) > 1e-3 * np.abs(D2[:, 0]).max()     # away from the zeros of R_1
    mean = (D3[far, 0] / D2[far, 0, None] ** 2 - 1).mean(0)
    say(f"[gpu] wide common error {dtype} P3={P3}: {float(np.abs(mean).max()):.1e}")
    assert far.sum() > 0.9 * n
    assert np.abs(mean).max() <= tol

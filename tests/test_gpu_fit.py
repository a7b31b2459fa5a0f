"""Linear fit on the device (pod_fit_gram, pod_fit_solve) against the fit
oracle (Sec. IV.A, eq. (63a); weights as in eq. (63b)).

Gram matrix: FP64 sums of up to ~10^4 products per entry, compared normwise
at 1e-12.  Solve: on well-conditioned random problems the coefficients
match the oracle's orthogonal solve to 1e-10; on POD descriptor matrices the
normal equations square the condition number (measured: 2e8 for the
21-descriptor set, 9e12 for the 103-descriptor set after diagonal scaling),
so the recovered coefficients are checked at 1e-6 for the former, and only
the fitted energies and forces (which the conditioning does not amplify) for
the latter."""
import numpy as np
import pytest
import torch

from gpu_common import oracle_params, say
from oracle import fit_oracle as fo
from oracle import pod_oracle as po
from paper_2212_14446_amd import pod, workloads as wl

pytestmark = pytest.mark.gpu

S = wl.PodSetup(0.5, 5.0, 8, 4, 4, 4, 3, 3)


def _h():
    return pod.PodModel(pod.setup_from_workload(S), "f64")


def _dev(x):
    return torch.as_tensor(np.ascontiguousarray(x, dtype=np.float64), device="cuda")


def _gram(m, G, E, dG, F, w_e, w_f, Z=None, accumulate=False):
    M = (G if G is not None and G.size else dG).shape[1]
    if Z is None:
        Z = torch.full((M + 1, M + 1), np.nan, dtype=torch.float64, device="cuda")
    n_cfg = 0 if G is None else G.shape[0]
    n_f = 0 if dG is None else dG.shape[0]
    pod.pod_fit_gram(m.h, M, n_cfg, None if n_cfg == 0 else _dev(G), None if n_cfg == 0 else _dev(E), w_e,
                     n_f, None if n_f == 0 else _dev(dG), None if n_f == 0 else _dev(F), w_f, Z, accumulate)
    pod.pod_check(m.h)
    return Z


def _problem(seed, n_cfg, R, M, scale=10.0):
    rng = np.random.default_rng(seed)
    return (rng.normal(size=(n_cfg, M)) * scale, rng.normal(size=n_cfg) * scale,
            rng.normal(size=(R, M)), rng.normal(size=R))


@pytest.mark.parametrize("M,n_cfg,R", [(103, 37, 10007), (21, 200, 4093), (1, 3, 17), (15, 5, 64),
                                       (16, 1, 1), (127, 9, 2051), (40, 0, 999), (40, 11, 0)])
def test_gram_matches_oracle(M, n_cfg, R):
    say(f"[gpu] fit gram M={M} n_cfg={n_cfg} R={R}")
    m = _h()
    G, E, dG, F = _problem(M + R, n_cfg, R, M)
    Z = _gram(m, G, E, dG, F, 100.0, 1.0).cpu().numpy()
    A, b = fo.design_matrix(G, dG, E, F, 100.0, 1.0)
    ref = fo.gram(A, b)
    assert np.all(Z == Z.T)
    assert np.abs(Z - ref).max() <= 1e-12 * np.abs(ref).max()


def test_gram_accumulate_and_reproducible():
    m = _h()
    G, E, dG, F = _problem(5, 30, 5000, 103)
    whole = _gram(m, G, E, dG, F, 100.0, 1.0)
    again = _gram(m, G, E, dG, F, 100.0, 1.0)
    assert torch.equal(whole, again)
    Z = _gram(m, G[:10], E[:10], dG[:1234], F[:1234], 100.0, 1.0)
    Z = _gram(m, G[10:], E[10:], dG[1234:], F[1234:], 100.0, 1.0, Z=Z, accumulate=True)
    ref = whole.cpu().numpy()
    assert np.abs(Z.cpu().numpy() - ref).max() <= 1e-13 * np.abs(ref).max()


@pytest.mark.parametrize("M,gamma", [(103, 0.0), (103, 1e-3), (21, 5.0), (1, 0.0), (127, 1e-12)])
def test_solve_matches_oracle(M, gamma):
    say(f"[gpu] fit solve M={M} gamma={gamma}")
    m = _h()
    G, E, dG, F = _problem(M, 50, 20 * M + 7, M)
    A, b = fo.design_matrix(G, dG, E, F, 100.0, 1.0)
    Z = _dev(fo.gram(A, b))
    c = torch.empty(M, dtype=torch.float64, device="cuda")
    loss = torch.empty(1, dtype=torch.float64, device="cuda")
    pod.pod_fit_solve(m.h, M, Z, gamma, c, loss)
    pod.pod_check(m.h)
    ref = fo.ridge_solve(A, b, gamma)
    got = c.cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-10 * np.abs(ref).max()
    f = fo.objective(A, b, ref, gamma)
    # the loss from the Gram blocks cancels b^T b against c^T A^T b
    assert abs(loss.item() - f) <= 1e-9 * float(b @ b)


def test_solve_singular_is_reported():
    m = _h()
    M = 7
    Z = torch.zeros((M + 1, M + 1), dtype=torch.float64, device="cuda")
    c = torch.full((M,), 5.0, dtype=torch.float64, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    pod.pod_fit_solve(m.h, M, Z, 0.0, c, loss)
    with pytest.raises(pod.PodError) as e:
        pod.pod_check(m.h)
    assert pod.ERRORS[e.value.code] == "POD_ESINGULAR"
    assert torch.all(c == 0) and torch.isnan(loss).all()
    # rank-deficient rows become solvable with gamma > 0
    G, E, dG, F = _problem(8, 3, 2, M)   # 5 rows < 7 unknowns
    A, b = fo.design_matrix(G, dG, E, F, 1.0, 1.0)
    pod.pod_fit_solve(m.h, M, _dev(fo.gram(A, b)), 0.1, c, loss)
    pod.pod_check(m.h)
    ref = fo.ridge_solve(A, b, 0.1)
    assert np.abs(c.cpu().numpy() - ref).max() <= 1e-10 * np.abs(ref).max()


def test_argument_errors():
    m = _h()
    Z = torch.zeros((5, 5), dtype=torch.float64, device="cuda")
    x = torch.zeros((3, 4), dtype=torch.float64, device="cuda")
    y = torch.zeros(3, dtype=torch.float64, device="cuda")
    for args, code in (((0, 3, x, y, 1.0, 0, None, None, 1.0, Z), "POD_EINVAL"),
                       ((4, 3, x, y, -1.0, 0, None, None, 1.0, Z), "POD_EINVAL"),
                       ((4, 3, None, y, 1.0, 0, None, None, 1.0, Z), "POD_EINVAL"),
                       ((4, 0, None, None, 1.0, 3, None, y, 1.0, Z), "POD_EINVAL"),
                       ((200, 3, x, y, 1.0, 0, None, None, 1.0, Z), "POD_ENOTSUP")):
        with pytest.raises(pod.PodError) as e:
            pod.pod_fit_gram(m.h, *args)
        assert pod.ERRORS[e.value.code] == code
    with pytest.raises(pod.PodError) as e:
        pod.pod_fit_solve(m.h, 4, Z, -1.0, y)
    assert pod.ERRORS[e.value.code] == "POD_EINVAL"


def _oracle_rows(b, s):
    p = oracle_params(s)
    Q, _ = po.pod_basis(p)
    G, dG = [], []
    for k in range(b.n_cfg):
        pos, cell, nl = b.config(k)
        args = (pos, cell, nl.offsets.astype(np.int64), nl.nbr_j, nl.shift3, p, Q)
        G.append(po.descriptors_fast(*args).sum(0))
        dG.append(po.global_descriptor_derivatives(*args).reshape(-1, s.M))
    return np.array(G), np.vstack(dG), Q


@pytest.mark.parametrize("setup,c_tol", [(wl.SETUP_CFG1, 1e-6), (wl.SETUP_CFG2, None)])
def test_fit_from_assembled_matrix(setup, c_tol):
    """Assemble D, G, dG/dR on the device, fit to labels made by the oracle
    from a known c, and recover c (or, where the matrix is too ill-conditioned
    for that, the labels)."""
    b = wl.make_batch(12, 31, setup, n_min=2, n_max=30)
    say(f"[gpu] fit end to end: M={setup.M} cells={b.n_cfg} atoms={b.N}")
    Go, dGo, Q = _oracle_rows(b, setup)
    c_true = wl.coefficients(setup.M, 3)
    E, F = Go @ c_true, -dGo @ c_true
    m = pod.PodModel(pod.setup_from_workload(setup), "f64", Q=Q[:, :max(setup.K2, setup.K3, setup.K4)])
    out = pod.batch_assemble(m, pod.DeviceBatch.from_batch(b), D=False)
    Gd, dGd = out["G"], out["dGdR"]
    M = setup.M
    Z = torch.empty((M + 1, M + 1), dtype=torch.float64, device="cuda")
    pod.pod_fit_gram(m.h, M, b.n_cfg, Gd, _dev(E), 100.0, 3 * b.N, dGd, _dev(F), 1.0, Z)
    c = torch.empty(M, dtype=torch.float64, device="cuda")
    loss = torch.empty(1, dtype=torch.float64, device="cuda")
    pod.pod_fit_solve(m.h, M, Z, 1e-12, c, loss)
    pod.pod_check(m.h)
    got = c.cpu().numpy()
    A, bb = fo.design_matrix(Go, dGo, E, F, 100.0, 1.0)
    pred, ref_pred = A @ got, A @ fo.ridge_solve(A, bb, 1e-12)
    assert np.linalg.norm(pred - bb) <= 1e-6 * np.linalg.norm(bb)
    assert np.linalg.norm(pred - ref_pred) <= 1e-6 * np.linalg.norm(bb)
    assert loss.item() <= 1e-10 * float(bb @ bb)
    if c_tol is not None:
        assert np.abs(got - c_true).max() <= c_tol * np.abs(c_true).max()


@pytest.mark.parametrize("M", [2, 15, 16, 17, 31, 48, 63, 64, 65, 95, 112, 128])
def test_solve_panel_edges(M):
    """Sizes around the 16-column panels, the 64 rows a lane holds of the back
    substitution, and the largest size; a diagonally scaled random problem
    (condition below 1e3), so the normal equations agree with the oracle's
    orthogonal solve to 1e3 x 128 x 2^-52 = 3e-11 at worst."""
    say(f"[gpu] fit solve panel edge M={M}")
    m = _h()
    G, E, dG, F = _problem(100 + M, 40, 20 * M + 7, M)
    A, b = fo.design_matrix(G, dG, E, F, 10.0, 1.0)
    c = torch.empty(M, dtype=torch.float64, device="cuda")
    loss = torch.empty(1, dtype=torch.float64, device="cuda")
    pod.pod_fit_solve(m.h, M, _dev(fo.gram(A, b)), 1e-3, c, loss)
    pod.pod_check(m.h)
    ref = fo.ridge_solve(A, b, 1e-3)
    assert np.abs(c.cpu().numpy() - ref).max() <= 1e-10 * np.abs(ref).max()
    assert abs(loss.item() - fo.objective(A, b, ref, 1e-3)) <= 1e-9 * float(b @ b)

"""Molecular dynamics on the device (pod_md_verlet, pod_md_max_displacement,
the md.MD driver with a device-built skin list) against the velocity-Verlet
oracle with POD oracle forces on an exact list at every step.

FP64 tolerance: the two sides differ only by summation order in the forces
(~1e-15 relative per step); over 20 steps of a smooth, gentle potential the
difference stays below 1e-10 relative, checked at 1e-9."""
import numpy as np
import pytest
import torch

from gpu_common import oracle_params, relerr, say
from oracle import md_oracle as mo
from oracle import pod_oracle as po
from paper_2212_14446_amd import md, pod, workloads as wl

pytestmark = pytest.mark.gpu

S = wl.PodSetup(0.5, 5.0, 6, 3, 3, 2, 2, 2)


def _system(n=2, seed=5, vscale=0.005, cscale=0.02):
    pos, cell = wl.bcc(n)
    pos = wl.displace(pos, 0.05, seed)
    c = cscale * wl.coefficients(S.M, seed + 1)
    vel = np.random.default_rng(seed + 2).normal(0.0, vscale, size=pos.shape)
    vel -= vel.mean(0)
    return pos, cell, vel, c


def _model(dtype="f64"):
    p = oracle_params(S)
    Q, _ = po.pod_basis(p)
    return pod.PodModel(pod.setup_from_workload(S), dtype, Q=Q[:, :p.K]), p, Q


def test_verlet_matches_oracle():
    pos, cell, vel, c = _system()
    m, p, Q = _model()
    dyn = md.MD(m, pos, vel, cell, c, skin=0.5)
    ep, ek = dyn.run(20, chunk=7, dt=1.0)
    x, v, oep, oek = mo.velocity_verlet(pos, vel, md.MASS_TA, 1.0, 20, mo.pod_force_fn(cell, p, Q, c))
    say(f"[gpu] md vs oracle: rebuilds {dyn.rebuilds}")
    assert relerr(dyn.x.cpu().numpy() - pos, x - pos) <= 1e-9
    assert relerr(dyn.v.cpu().numpy(), v) <= 1e-9
    assert relerr(ep.cpu().numpy(), oep[1:]) <= 1e-9
    assert relerr(ek.cpu().numpy(), oek[1:]) <= 1e-9


def test_rebuilds_momentum_and_energy():
    """Hot atoms force list rebuilds (and chunk retries); the trajectory
    equals one that rebuilds before every step, momentum is conserved and the
    total energy stays within the integrator's error."""
    pos, cell, vel, c = _system(3, seed=9, vscale=0.008)
    m, p, Q = _model()
    a = md.MD(m, pos, vel, cell, c, skin=0.15)
    ep, ek = a.run(120, chunk=10, dt=0.5)
    b = md.MD(m, pos, vel, cell, c, skin=0.15)
    for _ in range(120):
        b._rebuild()
        b.run(1, chunk=1, dt=0.5)
    say(f"[gpu] md rebuilds: {a.rebuilds} (every-step reference {b.rebuilds})")
    assert a.rebuilds > 2
    assert relerr(a.x.cpu().numpy() - pos, b.x.cpu().numpy() - pos) <= 1e-9
    mom0 = vel.sum(0)
    mom = a.v.cpu().numpy().sum(0)
    assert np.abs(mom - mom0).max() <= 1e-12 * max(1.0, np.abs(vel).sum())
    et = (ep + ek).cpu().numpy()
    e0 = float(ek[0].item())
    assert np.abs(et - et[0]).max() <= 1e-3 * e0


def test_fp32_follows_fp64():
    pos, cell, vel, c = _system(seed=11)
    m64, _, _ = _model("f64")
    m32, _, _ = _model("f32")
    a = md.MD(m64, pos, vel, cell, c)
    b = md.MD(m32, pos, vel, cell, c)
    a.run(20, dt=1.0)
    b.run(20, dt=1.0)
    dx = a.x.cpu().numpy() - pos
    assert relerr(b.x.double().cpu().numpy() - pos, dx) <= 1e-3


def test_max_displacement_and_errors():
    m, _, _ = _model()
    x = torch.zeros((5, 3), dtype=torch.float64, device="cuda")
    xr = torch.zeros_like(x)
    x[3, 1] = 0.25
    x[1, 0] = -0.1
    out = torch.empty(1, dtype=torch.float64, device="cuda")
    pod.pod_md_max_displacement(m.h, 5, x, xr, out)
    assert out.item() == 0.25
    x[2, 2] = float("nan")
    pod.pod_md_max_displacement(m.h, 5, x, xr, out)
    assert np.isnan(out.item())
    pos, cell, vel, c = _system()
    dyn = md.MD(m, pos, vel, cell, c)
    nb = dyn.nb
    args = (m.h, dyn.N, nb.P, dyn.x, dyn.v, dyn.F, cell, nb.offsets, nb.nbr_j, nb.shift, nb.rev, dyn.c)
    for mass, dt, extra in ((0.0, 1.0, {}), (180.0, float("nan"), {}), (180.0, 1.0, {"max_disp": out})):
        with pytest.raises(pod.PodError) as e:
            pod.pod_md_verlet(*args, mass, dt, 1, **extra)
        assert pod.ERRORS[e.value.code] == "POD_EINVAL"


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,nsteps", [(2, 1), (2, 3), (3, 66), (6, 5)])
def test_step_with_and_without_reverse_index(dtype, n, nsteps):
    """With a reverse index the kicks and the drift run inside the force
    gather; without one they are kernels of their own.  The two force sums
    differ in order only (32 terms at most here: 32 x 2^-53 relative in FP64
    of forces that move a step by 1e-3 of a unit), so trajectories agree to
    1e-11 (f64) and 2e-5 (f32, forces rounded to 2^-24 of a few eV/A)."""
    say(f"[gpu] md with/without reverse index n={n} steps={nsteps} {dtype}")
    import paper_2212_14446_amd.workloads as wl
    setup = wl.PodSetup(0.5, 5.0, 8, 4, 4, 4, 3, 3)
    m = pod.PodModel(pod.setup_from_workload(setup), dtype)
    rng = np.random.default_rng(17)
    base = np.stack(np.meshgrid(*[np.arange(n)] * 3, indexing="ij"), -1).reshape(-1, 3)
    pos = 3.3 * np.concatenate([base, base + 0.5]) + rng.normal(scale=0.05, size=(2 * n ** 3, 3))
    cell = 3.3 * n * np.eye(3)
    N = len(pos)
    x0 = torch.as_tensor(pos, dtype=m.torch_dtype, device="cuda")
    v0 = torch.as_tensor(rng.normal(scale=1e-3, size=(N, 3)), dtype=m.torch_dtype, device="cuda")
    c = torch.as_tensor(rng.normal(scale=1e-3, size=m.M), dtype=m.torch_dtype, device="cuda")
    nb = pod.DeviceNeighbors.build(m, x0, cell, rlist=5.4)
    nb.build_reverse(m)
    res = []
    for rev in (nb.rev, None):
        x, v = x0.clone(), v0.clone()
        F = m.energy_forces(x, cell, nb, c)["F"]
        ep = torch.empty(nsteps, dtype=torch.float64, device="cuda")
        ek = torch.empty_like(ep)
        disp = torch.empty(1, dtype=torch.float64, device="cuda")
        pod.pod_md_verlet(m.h, N, nb.P, x, v, F, cell, nb.offsets, nb.nbr_j, nb.shift, rev, c, 180.9, 1.0, nsteps,
                          ep, ek, x0, disp)
        m.check()
        res.append([t.double().cpu().numpy() for t in (x, v, F, ep, ek, disp)])
    tol = 1e-11 if dtype == "f64" else 2e-5
    for a, b in zip(*res):
        assert np.abs(a - b).max() <= tol * max(np.abs(b).max(), 1e-30)
    x = res[0][0]
    assert res[0][5][0] >= np.linalg.norm(x - x0.double().cpu().numpy(), axis=1).max() * (1 - 1e-12)

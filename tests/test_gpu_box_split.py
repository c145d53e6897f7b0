"""Box meshes whose velocity chunks are dealt to several workgroups per
element: FP64 steps against the oracle where each workgroup still walks eight
chunks (343 elements, p = 1), where the split is chosen by rounds (60 and 8
elements, a chunk count that no split divides), and with the reduced pair,
whose split runs across the two components.  Tolerance as for every FP64 step
(1e-12 relative L2)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,p,nv,model,rk,delta", [
    ((7, 7, 7), 1, (20, 13, 16), 0, 0, 0.0),
    ((5, 4, 3), 2, (13, 11, 9), 1, 1, 0.0),
    ((2, 2, 2), 3, (11, 13, 7), 1, 0, 0.0),
    ((2, 2, 2), 2, (11, 13, 7), 0, 1, 2.0),
])
def test_split_steps_match_oracle(orc, N, p, nv, model, rk, delta):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd.frdvm import FrDvm
    mesh, grid = W.box_mesh(N), W.grid_spec(nv, 5.0)
    par = {"model": model, "prandtl": 0.71 if model else 1.0, "mu_ref": 0.02, "theta_ref": 1.0, "omega": 0.81,
           "newton_tol": 1e-13, "newton_max_iter": 50}
    prim = W.prim_random_modes(W.box_solution_points(mesh, p), seed=3 + p, U_amp=0.3)
    f0 = W.maxwellian(prim, grid).numpy()
    rng = np.random.default_rng(9)
    f0 *= 1.0 + 0.02 * rng.uniform(-1, 1, f0.shape)
    if delta:
        g0 = 0.45 * delta * f0 * (1.0 + 0.02 * rng.uniform(-1, 1, f0.shape))
        f0 = np.concatenate([f0, g0], -1)
    P = orc.Problem(mesh, p, grid, dict(par, delta=delta) if delta else par)
    dt = P.dt(0.2)
    ref = P.rk_step(f0, dt, scheme=rk, nsteps=1)
    s = FrDvm(mesh, p, grid, dict(par, rk=rk), delta=delta)
    f = torch.as_tensor(f0).cuda().reshape(s.shape).contiguous()
    s.rk_step(f, dt)
    got = f.cpu().numpy().reshape(ref.shape)
    assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref)
    Q = torch.empty((s.ne * s.ns, 5), dtype=torch.float64, device="cuda")
    s.moments(f, Q)
    Qr = np.asarray(P.moments(ref)).reshape(-1, 5)
    assert np.linalg.norm(Q.cpu().numpy() - Qr) <= 1e-12 * np.linalg.norm(Qr)

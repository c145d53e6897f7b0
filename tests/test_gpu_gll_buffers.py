"""Gauss-Lobatto boxes step through the caller's buffer, the register and one
stage value.  Velocity grids with a single node of zero velocity in two
directions, where two buffers of traces are the smaller and are kept at p = 3,
and grids just on the other side of that line: residual, and steps of both
schemes one after the other on one handle, against the oracle (FP64, 1e-12)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("p", [1, 3])
@pytest.mark.parametrize("nv", [(64, 1, 1), (9, 3, 1), (3, 3, 3), (8, 8, 1)])
def test_small_traces(orc, p, nv):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd import frdvm as F
    umax = [5.0 if n > 1 else 0.0 for n in nv]
    grid = {"n": list(nv), "umin": [-u for u in umax], "umax": umax}
    mesh = W.box_mesh((3, 2, 2), length=(1.0, 0.8, 0.7))
    par = {"model": 2, "mu_ref": 1.0}
    P = orc.Problem(mesh, p, grid, dict(par, nodes=1))
    f0 = np.random.default_rng(p).uniform(0.5, 1.5, (mesh["n_elem"], (p + 1) ** 3, P.nu))
    s = F.FrDvm(mesh, p, grid, par, nodes=1)
    f = torch.as_tensor(f0).cuda().reshape(s.shape).contiguous()
    R = torch.empty_like(f)
    s.residual(f, R)
    ref = P.residual(f0)
    assert np.abs(R.cpu().numpy().reshape(ref.shape) - ref).max() <= 1e-12 * max(1.0, np.abs(ref).max())
    dt = P.dt(0.2)
    ref = P.rk_step(P.rk_step(f0, dt, scheme=1, nsteps=3), dt, scheme=0, nsteps=2)
    s.set_params(**dict(par, rk=1))
    s.rk_steps(f, dt, 3)
    s.set_params(**dict(par, rk=0))
    s.rk_steps(f, dt, 2)
    assert np.linalg.norm(f.cpu().numpy().reshape(ref.shape) - ref) <= 1e-12 * np.linalg.norm(ref)

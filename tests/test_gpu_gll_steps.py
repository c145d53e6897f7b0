"""Steps on boxes with Gauss-Lobatto points, whose stages read the inflow
traces from the neighbours' stage values, against the oracle on the same
points: orders 1 to 3, both schemes, several steps in one call and a change
of scheme between calls, ragged velocity grids with and without nodes of zero
velocity, directions of a single element (its own periodic neighbour), the
overlapped solve (same bits), the reduced pair, a batch with split elements,
and the move to the limiter's path.  FP64 to 1e-12 relative L2; FP32
deviation storage over four steps to the bounds it has on Gauss points (f
2e-7, moments 1.5e-7); FP32 to 12 stages' roundings of 2^-24 each (1e-6)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a) - np.asarray(b)) / np.linalg.norm(np.asarray(b)))


@pytest.fixture(scope="module")
def F():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd import frdvm
    frdvm.lib()
    return frdvm


def _case(orc, N, p, nv, model, delta, dtype=torch.float64):
    mesh, grid = W.box_mesh(N, length=(1.0, 0.8, 0.7)), W.grid_spec(nv, 5.0)
    par = {"model": model, "prandtl": 0.71 if model else 1.0, "mu_ref": 0.02, "theta_ref": 1.0, "omega": 0.81,
           "newton_tol": 1e-13, "newton_max_iter": 50}
    P = orc.Problem(mesh, p, grid, dict(par, nodes=1, **({"delta": delta} if delta else {})))
    prim = W.prim_random_modes(P.geo["xs"], seed=11 + p, U_amp=0.3)
    f0 = W.maxwellian(prim, grid).numpy()
    rng = np.random.default_rng(5 + p)
    f0 *= 1.0 + 0.03 * rng.uniform(-1.0, 1.0, f0.shape)
    if delta:
        f0 = np.concatenate([f0, 0.45 * delta * f0 * (1.0 + 0.02 * rng.uniform(-1, 1, f0.shape))], -1)
    if dtype != torch.float64:
        f0 = f0.astype(np.float32).astype(np.float64)
    return mesh, grid, par, P, f0


CASES = [
    ((3, 2, 2), 1, (9, 8, 7), 1, 0.0),
    ((1, 3, 2), 2, (7, 6, 5), 0, 0.0),
    ((3, 1, 1), 3, (6, 5, 4), 1, 0.0),
    ((1, 1, 1), 3, (3, 4, 5), 0, 0.0),
    ((2, 3, 2), 2, (7, 6, 5), 0, 2.0),
    ((2, 2, 2), 3, (11, 13, 7), 1, 2.0),
    ((2, 2, 2), 3, (16, 13, 11), 0, 0.0),
]


@pytest.mark.parametrize("N,p,nv,model,delta", CASES)
def test_fp64_steps(F, orc, N, p, nv, model, delta):
    mesh, grid, par, P, f0 = _case(orc, N, p, nv, model, delta)
    dt = P.dt(0.2)
    ref0 = P.rk_step(f0, dt, scheme=0, nsteps=2)
    ref = P.rk_step(ref0, dt, scheme=1, nsteps=2)
    outs = []
    for overlap in (0, 1):
        s = F.FrDvm(mesh, p, grid, dict(par, rk=0, overlap=overlap, guess=0), nodes=1, delta=delta)
        f = torch.as_tensor(f0).cuda().reshape(s.shape).contiguous()
        s.rk_steps(f, dt, 2)
        assert rel(f.cpu().numpy().reshape(ref.shape), ref0) < 1e-12
        s.set_params(**dict(par, rk=1, overlap=overlap, guess=0))
        s.rk_steps(f, dt, 2)
        assert rel(f.cpu().numpy().reshape(ref.shape), ref) < 1e-12
        outs.append(f)
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("N,p,nv,model,rk", [((3, 2, 2), 1, (9, 8, 7), 1, 0), ((3, 2, 2), 2, (9, 8, 7), 0, 1),
                                              ((3, 1, 2), 3, (9, 8, 7), 1, 0), ((3, 1, 2), 3, (9, 8, 7), 1, 1)])
def test_fp32_steps(F, orc, N, p, nv, model, rk):
    mesh, grid, par, P, f0 = _case(orc, N, p, nv, model, 0.0, torch.float32)
    dt = P.dt(0.2)
    ref = P.rk_step(f0, dt, scheme=rk, nsteps=4)
    Qr = P.moments(ref)
    for prec in (F.FP32_DEV, F.FP32):
        s = F.FrDvm(mesh, p, grid, dict(par, precision=prec, rk=rk, guess=1), nodes=1)
        f = torch.as_tensor(f0, dtype=torch.float32).cuda().reshape(s.shape).contiguous()
        s.rk_steps(f, dt, 4)
        got = f.double().cpu().numpy().reshape(ref.shape)
        Q = P.moments(got)
        eq = [rel(Q[..., 0], Qr[..., 0]), rel(Q[..., 1:4], Qr[..., 1:4]), rel(Q[..., 4], Qr[..., 4])]
        print(f"p {p} rk {rk} precision {prec}: f {rel(got, ref):.2e}, moments {[f'{x:.2e}' for x in eq]}", flush=True)
        if prec == F.FP32_DEV:
            assert rel(got, ref) < 2e-7 and max(eq) < 1.5e-7
        else:
            assert rel(got, ref) < 1e-6 and max(eq) < 1e-6


def test_move_to_the_limiters_path(F, orc):
    mesh, grid, par, P, f0 = _case(orc, (2, 2, 2), 2, (7, 6, 5), 0, 0.0)
    dt = P.dt(0.2)
    ref = P.rk_step(f0, dt, scheme=1, nsteps=1)
    ref = orc.Problem(mesh, 2, grid, dict(par, nodes=1, positivity=1)).rk_step(ref, dt, scheme=1, nsteps=1)
    s = F.FrDvm(mesh, 2, grid, dict(par, rk=1), nodes=1)
    f = torch.as_tensor(f0).cuda().reshape(s.shape).contiguous()
    s.rk_step(f, dt)
    s.set_params(**dict(par, rk=1, positivity=1))
    s.rk_step(f, dt)
    assert rel(f.cpu().numpy().reshape(ref.shape), ref) < 1e-12

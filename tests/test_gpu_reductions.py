"""Newton statistics and domain totals at point counts around the reductions'
workgroups (256 points, four per thread): the histogram counts every point
once and agrees with the per-point outcomes, totals are the weighted sums of
the returned moments (FP64 sums of up to 5184 terms: 1e-13)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,p,model", [((1, 1, 1), 1, 0), ((4, 4, 2), 1, 1), ((3, 11, 1), 1, 0), ((9, 8, 9), 1, 0),
                                       ((2, 2, 4), 3, 1)])
def test_statistics_and_totals(N, p, model):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd.frdvm import FrDvm
    mesh, grid = W.box_mesh(N), W.grid_spec((7, 6, 8), 5.0)
    s = FrDvm(mesh, p, grid, {"model": model, "prandtl": 0.8, "mu_ref": 0.05})
    prim = W.prim_random_modes(W.box_solution_points(mesh, p), seed=2, U_amp=0.4)
    prim[0, 0, 0] = -1.0  # a point without an equilibrium
    f = W.maxwellian(prim, grid).cuda().reshape(s.shape).contiguous()
    s.newton_stats(reset=True)
    s.collide(f, torch.empty_like(f))
    st, (status, iters, resid) = s.newton_stats(reset=True), s.newton_points()
    status, iters, resid = (t.cpu().numpy().reshape(-1) for t in (status, iters, resid))
    assert np.array_equal(st["hist"], np.bincount(np.clip(iters, 0, 63), minlength=64))
    assert st["n_fallback"] == (status == 1).sum() and st["n_guard"] == (status == 3).sum()
    assert st["max_resid"] == max(0.0, resid[np.isfinite(resid)].max())
    Q = torch.empty((s.ne * s.ns, 5), dtype=torch.float64, device="cuda")
    tot = s.moments(f, Q, totals=True)
    wq = np.polynomial.legendre.leggauss(p + 1)[1]
    w = np.einsum("k,j,i->kji", wq, wq, wq).reshape(-1) / 8.0 / mesh["n_elem"]
    Q = Q.cpu().numpy().reshape(s.ne, s.ns, 5)
    scale = np.abs(Q * w[None, :, None]).sum((0, 1))
    assert np.all(np.abs(tot - (Q * w[None, :, None]).sum((0, 1))) <= 1e-13 * scale)

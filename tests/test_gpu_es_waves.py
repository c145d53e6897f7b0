"""ES Newton, a wave per point's sums: grids on both sides of every lane
layout (64 / n_x lanes per x node; y counts that the lanes' strides do not
divide; more y and z nodes than lanes) and point counts with 4, 16 and 64
points per workgroup, the last workgroup partial, against the oracle on a few
strongly anisotropic states repeated over the points; a point without an
equilibrium among them.  FP64 tolerance of the collision tests (1e-12 of the
equilibrium), for the factorised and the direct sums alike."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _states(P, n, seed):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(n):
        Lm = np.eye(3) + 0.35 * rng.uniform(-1, 1, (3, 3))
        c = (P.u - rng.uniform(-0.6, 0.6, 3)) @ Lm
        f = rng.uniform(0.5, 2.0) * np.exp(-0.5 * (c * c).sum(1) / rng.uniform(0.8, 1.3))
        out.append(f * rng.uniform(0.8, 1.2, P.nu))
    return np.array(out)


def _check(orc, N, p, nv, direct, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd import frdvm
    monkeypatch.setenv("FRDVM_ES_DIRECT", "1" if direct else "0")
    grid = W.grid_spec(nv, (5.0, 4.5, 5.5))
    par = {"model": 1, "prandtl": 2.0 / 3.0, "mu_ref": 0.05}
    P = orc.Problem.points_only(grid, par)
    f5 = _states(P, 5, sum(nv))
    ref = P.collide(f5)
    h = frdvm.FrDvm(W.box_mesh(N), p, grid, par)
    n = h.ne * h.ns
    i = np.arange(n) % 5
    f = torch.as_tensor(f5).cuda()[torch.as_tensor(i).cuda()].clone()
    bad = n - 2
    f[bad] = 0.0
    f = f.reshape(h.shape).contiguous()
    S, Qp = torch.empty_like(f), torch.empty((n, 5), dtype=torch.float64, device="cuda")
    h.collide(f, S, Qp)
    status = h.newton_points()[0].reshape(-1).cpu().numpy()
    assert status[bad] == frdvm.NEWTON_NONREAL
    assert np.array_equal(np.delete(status, bad), np.delete(np.asarray(ref[3])[i], bad))
    S, Qp = S.reshape(n, -1), Qp.cpu().numpy()
    for k in range(5):
        rows = np.nonzero((i == k) & (np.arange(n) != bad))[0]
        got = S[torch.as_tensor(rows).cuda()]
        assert torch.equal(got, got[:1].expand_as(got))  # the same bits wherever the point sits
        # (S = (g - f) / tau is some tenths of its terms: ten times the tolerance of g)
        assert np.linalg.norm(got[0].cpu().numpy() - ref[0][k]) <= 1e-11 * np.linalg.norm(ref[0][k])
        assert np.abs(Qp[rows[0]] - ref[1][k]).max() <= 1e-12 * max(1.0, np.abs(ref[1][k]).max())


@pytest.mark.parametrize("direct", [False, True])
@pytest.mark.parametrize("nv", [(8, 9, 7), (16, 16, 16), (19, 17, 18), (21, 7, 40), (22, 23, 9), (32, 11, 8),
                                (33, 8, 9), (64, 6, 7), (10, 64, 33), (7, 8, 64)])
def test_grids(orc, nv, direct, monkeypatch):
    _check(orc, (3, 2, 1), 2, nv, direct, monkeypatch)


@pytest.mark.parametrize("N,p", [((1, 1, 1), 1), ((9, 10, 3), 3), ((32, 33, 1), 3)])
def test_point_counts(orc, N, p, monkeypatch):
    _check(orc, N, p, (9, 7, 8), False, monkeypatch)

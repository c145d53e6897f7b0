"""The BGK Newton kernel gives a point 1, 2, 4 or 8 lanes by the batch size:
the same few states repeated to batches on both sides of every line (axis of
12 nodes: 1536, 6144, 24576 points) have the oracle's root in every row
(1e-10, as for the training targets), on a ragged grid with axes shorter than
the lanes, and a point without an equilibrium is marked in each."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 9, 1536, 1537, 6144, 6145, 24576, 24577])
def test_every_lane_count_finds_the_root(orc, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd import frdvm
    grid = W.grid_spec((12, 7, 9), (5.0, 4.0, 4.5))
    par = {"model": 0, "mu_ref": 1.0}
    h = frdvm.FrDvm(W.box_mesh(1), 1, grid, par)
    P = orc.Problem.points_only(grid, par)
    rng = np.random.default_rng(8)
    f = np.exp(-0.5 * ((P.u - [0.4, -0.3, 0.2]) ** 2).sum(1) / 0.9)[None] * rng.uniform(0.6, 1.4, (5, P.nu))
    Q, zr = orc.moments(f, P.u, P.w), P.collide(f)[2]
    i = np.arange(n) % 5
    Qn = Q[i].copy()
    Qn[n // 2] = [-1.0, 0, 0, 0, 1.0]
    z, it, ev, st, res = (t.cpu().numpy() for t in h.equilibrium(torch.as_tensor(Qn).cuda().contiguous()))
    ok = np.arange(n) != n // 2
    assert st[n // 2] == frdvm.NEWTON_NONREAL and np.all(z[n // 2] == 0)
    assert np.all(st[ok] == 0) and np.all(it[ok] > 0) and np.all(ev[ok] > 0)
    if ok.any():
        assert np.abs(z - zr[i])[ok].max() < 1e-10


def test_solve_of_a_part_sums_like_the_whole():
    """8 x 5 x 4 elements at p = 1 (1280 points, 8-node axes): the halves of an
    overlapped solve lie below a line (1024 points) that the whole lies above;
    steps give the same bits either way."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd import frdvm
    mesh, grid = W.box_mesh((8, 5, 4)), W.grid_spec(8, 5.0)
    f0 = W.maxwellian(W.prim_random_modes(W.box_solution_points(mesh, 1), seed=4, U_amp=0.3), grid)
    out = []
    for overlap in (0, 1):
        s = frdvm.FrDvm(mesh, 1, grid, {"model": 0, "mu_ref": 0.02, "overlap": overlap})
        f = f0.cuda().reshape(s.shape).contiguous()
        s.rk_steps(f, s.dt(0.2), 2)
        out.append(f)
    assert torch.equal(*out)

"""ES Newton, the factorised sums at the end of their range: thin ridges
across coarse velocity grids whose y axis is padded to the lanes' stride
(8 x 9, 4 x 17, 5 x 13 nodes in x and y: up to twice the axis), where a row's
factor goes on growing in the padded nodes.  Every state has an equilibrium by
the direct sums; the factorised form has to find one too, with a final
residual at the rounding floor (a hundred times the tolerance).

And cold, sheared states on wide grids, whose cross exponents lie between the
reach of the factorised form and twice that: the wide form of the sums against
the direct one (status, evaluations, Q' to 1e-9: the root's condition, some
1e4, times the tolerance 1e-13), for every sign of the shear, grids that the
lanes' strides do and do not divide, and at a time well below that of the
direct sums."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# widths along, across the ridge and in z, and its angle to the x axis
RIDGES = {
    ((8, 9, 7), (3.0, 10.0, 4.0), 2 / 3): [(1.9456662955560242, 0.2998534103984082, 0.3830887157424361, 0.3209881557597111),
                                           (2.688391305941946, 0.23566465669188533, 0.3685365526331489, 2.8352904448110987)],
    ((8, 9, 7), (6.0, 20.0, 20.0), 2 / 3): [(6.542660959648983, 0.413235150073954, 0.3724483055529204, 0.5493212049578771),
                                            (3.629749821979678, 0.2964304818052859, 1.8609330015804482, 2.5058079574763283)],
    ((4, 17, 8), (3.0, 6.0, 4.0), 0.5): [(0.9673133260576533, 0.40275117533074395, 0.9543570438799283, 0.7376083540961491),
                                         (0.6362029039351752, 0.213229032586413, 0.9792677910071045, 2.76357447408688)],
    ((5, 13, 9), (3.0, 10.0, 4.0), 2 / 3): [(2.2619707791714605, 0.16861909064288494, 0.40059367313158234, 0.2886247031446031),
                                            (2.623911440589854, 0.31112147708322707, 0.38074988198523674, 2.883944349673468)],
}


@pytest.mark.parametrize("key", list(RIDGES))
def test_padded_rows(key, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd import frdvm as F
    nv, um, pr = key
    grid = W.grid_spec(nv, um)
    ax = [np.linspace(-um[d], um[d], nv[d]) for d in range(3)]
    u = np.stack(np.meshgrid(ax[2], ax[1], ax[0], indexing="ij"), -1)[..., ::-1].reshape(-1, 3)
    f = []
    for s1, s2, s3, a in RIDGES[key]:
        v = np.array([np.cos(a) * um[0], np.sin(a) * um[1]])
        v /= np.linalg.norm(v)
        al, ac = u[:, :2] @ v, u[:, 0] * v[1] - u[:, 1] * v[0]
        f.append(np.exp(-0.5 * ((al / s1) ** 2 + (ac / s2) ** 2 + (u[:, 2] / s3) ** 2)) + 1e-12)
    f = np.array(f)[np.arange(8) % len(f)]
    for direct in ("1", "0"):
        monkeypatch.setenv("FRDVM_ES_DIRECT", direct)
        h = F.FrDvm(W.box_mesh(1), 1, grid, {"model": 1, "prandtl": pr, "mu_ref": 1e-2, "newton_max_iter": 100})
        fg = torch.as_tensor(f).cuda().reshape(h.shape).contiguous()
        S, Qp = torch.empty_like(fg), torch.empty((8, 5), dtype=torch.float64, device="cuda")
        h.collide(fg, S, Qp)
        status, _, res = (t.cpu().numpy().reshape(-1) for t in h.newton_points())
        print(f"direct {direct}: status {status.tolist()}, residual {res.max():.1e}", flush=True)
        assert np.all(status == F.NEWTON_OK), (direct, status)
        assert res.max() <= 1e-11 and torch.isfinite(S).all() and torch.isfinite(Qp).all()


def _sheared(n, um, e, d, U):
    """Gaussian of covariance e I + (3 - 3 e) d d^T (trace 3) about U on the nodes."""
    ax = [torch.linspace(-um[k], um[k], n[k], dtype=torch.float64, device="cuda") - U[k] for k in range(3)]
    u = torch.stack(torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij"), -1).flip(-1).reshape(-1, 3)
    d = torch.tensor(d, dtype=torch.float64, device="cuda")
    d = d / d.norm()
    C = e * torch.eye(3, dtype=torch.float64, device="cuda") + (3 - 3 * e) * torch.outer(d, d)
    return torch.exp(-0.5 * ((u @ torch.linalg.inv(C)) * u).sum(1))


SIGNS = [(1, 1, 1), (-1, 1, 1), (1, -1, 1), (1, 1, -1), (1, 1, 0), (1, -1, 0), (0, 1, 1), (1, 0, -1)]


@pytest.mark.parametrize("n,um,e", [((20, 20, 20), (8.0, 8.0, 8.0), 0.1), ((19, 17, 18), (8.0, 7.5, 8.5), 0.1),
                                    ((33, 21, 15), (8.0, 8.0, 7.0), 0.08), ((10, 33, 21), (6.0, 8.0, 8.0), 0.1),
                                    ((24, 24, 25), (12.0, 12.0, 12.0), 0.2)])
def test_wide_form_equals_direct_sums(n, um, e, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd import frdvm as F
    f = torch.stack([_sheared(n, um, e, d, (0.3, -0.2, 0.4)) for d in SIGNS])
    out = []
    for direct in ("1", "0"):
        monkeypatch.setenv("FRDVM_ES_DIRECT", direct)
        h = F.FrDvm(W.box_mesh(1), 1, W.grid_spec(n, um), {"model": 1, "prandtl": 2 / 3, "mu_ref": 1e-2, "newton_max_iter": 100})
        fg = f.reshape(h.shape).contiguous()
        S, Qp = torch.empty_like(fg), torch.empty((8, 5), dtype=torch.float64, device="cuda")
        h.collide(fg, S, Qp)
        status, its, res = h.newton_points()
        assert int(status.abs().max()) == F.NEWTON_OK and float(res.max()) <= 1e-11
        out.append((its, Qp))
    print("steps", out[0][0].flatten().tolist(), "Q' differs by", float((out[0][1] - out[1][1]).abs().max()), flush=True)
    assert torch.equal(out[0][0], out[1][0])
    assert torch.allclose(out[0][1], out[1][1], rtol=1e-9, atol=1e-9)


def test_wide_form_is_taken(monkeypatch):
    """13,824 points with exponents between the two forms' ranges: the solve
    takes less than half the time of the direct sums (measured: a fifth)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2312_06567_amd import frdvm as F
    n, um = (20, 20, 20), (8.0, 8.0, 8.0)
    t = []
    for direct in ("1", "0"):
        monkeypatch.setenv("FRDVM_ES_DIRECT", direct)
        h = F.FrDvm(W.box_mesh(12), 1, W.grid_spec(n, um), {"model": 1, "prandtl": 2 / 3, "mu_ref": 1e-2, "newton_max_iter": 100})
        f = _sheared(n, um, 0.15, (1, 1, 1), (0.0, 0.0, 0.0)).repeat(h.ne * h.ns, 1).reshape(h.shape).contiguous()
        S = torch.empty_like(f)
        h.collide(f, S)
        h.profile_read(reset=True)
        h.profile(True)
        for _ in range(5):
            h.collide(f, S)
        h.profile(False)
        ms, launches = h.profile_read(reset=True)["newton"]
        t.append(ms / launches)
        del f, S
    print(f"solve: direct {t[0]:.3f} ms, factorised {t[1]:.3f} ms", flush=True)
    assert t[1] < 0.5 * t[0]

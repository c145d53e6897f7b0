"""Prisms and tetrahedra in FP32: the residual of a state uniform in space
(values with random mantissas, one per velocity) is rounding error alone, the
part of it that grows with the order.  The kernels form the derivatives at the
points of degree p - 1 and interpolate them; in root mean square the error may
not exceed that of the dense derivative matrices applied in FP32, entry after
entry in fused multiply-adds (emulated here on the oracle's operators)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
f32 = np.float32


def _fma(a, b, c):
    return (np.float64(a) * np.float64(b) + np.float64(c)).astype(f32)


def _dense_error(D, c, f):
    """-sum_a c_a D_a f of the constant f (per velocity), [points, velocities]."""
    D = np.where(np.abs(D) < 1e-12, 0.0, D).astype(f32)
    r = np.zeros((D.shape[1], f.size), f32)
    for a in range(3):
        for i in range(D.shape[1]):
            g = np.zeros(f.size, f32)
            for j in np.nonzero(D[a, i])[0]:
                g = _fma(D[a, i, j], f, g)
            r[i] = _fma(-c[a], g, r[i])
    return r


@pytest.mark.parametrize("p", [1, 2, 3])
def test_no_more_error_than_the_dense_operators(p):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import mixed as M
    from paper_2312_06567_amd import frdvm as F
    mesh, grid = W.prism_tet_box_mesh(3), W.grid_spec((9, 8, 7), 5.0)
    s = F.FrDvm(mesh, p, grid, {"model": 2, "mu_ref": 1.0, "precision": F.FP32})
    val = np.random.default_rng(p).uniform(1.0, 2.0, s.nu).astype(f32)
    f = torch.as_tensor(val).cuda().repeat(s.ne, 1).reshape(s.shape).contiguous()
    R = torch.empty_like(f)
    s.residual(f, R)
    R = R.cpu().numpy().reshape(-1, s.nu)
    ax = [np.linspace(-5.0, 5.0, n) for n in grid["n"]]
    u = np.stack(np.meshgrid(ax[2], ax[1], ax[0], indexing="ij"), -1)[..., ::-1].reshape(-1, 3)
    et = np.asarray(mesh["elem_type"])
    first = np.concatenate([[0], np.cumsum([M.ref_element(int(t), p).ns for t in et])])
    for t, name in ((M.PRISM, "prisms"), (M.TET, "tetrahedra")):
        ref = M.ref_element(t, p)
        got = want = 0.0
        for e in np.nonzero(et == t)[0][::7]:
            v = mesh["nodes"][mesh["elem_nodes"][e][:M.NVERT[t]]]
            grad = np.linalg.inv(0.5 * np.stack([v[a] - v[0] for a in M.AXES[t]], 1))  # rows: grad xi_a
            want += (_dense_error(np.array(ref.D), (u @ grad.T).T.astype(f32), val).astype(float) ** 2).sum()
            got += (R[first[e]:first[e + 1]].astype(float) ** 2).sum()
        print(f"p {p} {name}: error {np.sqrt(got):.3e}, dense operators {np.sqrt(want):.3e}", flush=True)
        assert got <= want

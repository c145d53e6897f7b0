"""Cases that the speed of this framework is measured on.

Each is work that a program using the framework has it do, through the public
binding (``FrDvm``, ``Mlp``), over the range of sizes, meshes, storage forms
and gas models that the repository's workloads and tests use:

  step         explicit Runge-Kutta steps (the solver's main loop) on a periodic
               box, a curved O-grid with wall and farfield, or a prism /
               tetrahedron box, the state advanced in place
  operators    residual and collision source as separate calls, for a program
               with its own time integrator
  diagnostics  moments, domain totals and the local Knudsen number of a state
  equilibrium  conservative equilibria of a batch of macroscopic states
  train        one optimiser step of the learned Newton start
  predict      its forward pass

``exact`` gives the same results in 64 bits from plain torch / numpy: the
flux-reconstruction residual through element-local dense or line operators,
the conservative equilibrium through an undivided Newton iteration on sums
over the whole velocity grid.
"""
import math

import numpy as np
import torch

import workloads
from paper_2312_06567_amd import frdvm

SSP, LSRK = 0, 1
BGK, ES = 0, 1
F64, F32, DEV = 0, 1, 2
H_NET = 64


# ------------------------------------------------------------------- cases --

def _step(name, mesh, size, p, nv, umax, model, precision, rk, nodes=0, delta=0.0, kn=1e-3, steps=1, kind="step"):
    return {"name": name, "kind": kind, "mesh": mesh, "nx": size[0], "ny": size[1], "nz": size[2], "p": p,
            "n0": nv[0], "n1": nv[1], "n2": nv[2], "umax": float(umax), "model": model, "precision": precision,
            "rk": rk, "nodes": nodes, "delta": float(delta), "kn": float(kn), "steps": steps}


def listed():
    return [
        # the smallest workload of the repository: a step that is all launches and latency
        _step("box4_p1_v8_bgk_f64", "box", (4, 4, 4), 1, (8, 8, 8), 6.0, BGK, F64, SSP, kn=0.05),
        # the ragged velocity grid of the parity tests on a small odd box, several steps a call
        _step("box5x4x3_p2_v19x17x18_es_f32", "box", (5, 4, 3), 2, (19, 17, 18), 8.0, ES, F32, LSRK, steps=2),
        # the mid-size FP64 workload (16^3 elements, 16^3 velocities)
        _step("box16_p3_v16_bgk_f64", "box", (16, 16, 16), 3, (16, 16, 16), 6.0, BGK, F64, SSP),
        # the benchmark's form (ES-BGK, deviation storage, low-storage scheme) on a mesh that fits three times
        _step("box16_p3_v20_es_dev", "box", (16, 16, 16), 3, (20, 20, 20), 8.0, ES, DEV, LSRK, kn=2e-4),
        # what the benchmark compares it with: plain FP64, SSP-RK3
        _step("box12_p3_v20_es_f64", "box", (12, 12, 12), 3, (20, 20, 20), 8.0, ES, F64, SSP, kn=2e-4),
        # Mach-8 flow past a cylinder: curved elements, diffuse wall, farfield, positivity limiter
        _step("ogrid48x24x2_p2_v24_es_f32", "ogrid", (48, 24, 2), 2, (24, 24, 24), 14.0, ES, F32, LSRK, kn=0.01),
        # the paper's element types at its velocity resolution
        _step("ptbox8_p3_v24_es_f32", "ptbox", (8, 8, 8), 3, (24, 24, 24), 8.0, ES, F32, LSRK),
        # gas with internal energy: the reduced pair of distributions
        _step("box6_p3_v16_es_f32_pair", "box", (6, 6, 6), 3, (16, 16, 16), 8.0, ES, F32, SSP, delta=2.0),
        # a program with its own integrator: residual and collision as calls, Gauss-Lobatto points
        _step("operators_box8_p3_v16_es_f64", "box", (8, 8, 8), 3, (16, 16, 16), 7.0, ES, F64, SSP, nodes=1,
              kind="operators"),
        # monitoring of a run: moments, totals and the continuum-breakdown field
        _step("diagnostics_box16_p3_v16_f32", "box", (16, 16, 16), 3, (16, 16, 16), 6.0, BGK, F32, SSP,
              kind="diagnostics"),
        # training targets and evaluation of the learned start: a batch of states on the 32^3 grid
        {"name": "equilibrium_65536_v32_learned", "kind": "equilibrium", "n": 65536, "nv": 32, "umax": 10.0, "guess": 2},
        # the learned start's training step at its default batch and width
        {"name": "train_b4096_h64", "kind": "train", "batch": 4096, "hidden": 64},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["box", "box", "box", "ogrid", "ptbox", "operators", "diagnostics", "equilibrium", "train",
                       "predict"])
    if kind == "equilibrium":
        return {"kind": kind, "n": _logint(rng, 1000, 100000), "nv": rng.choice([16, 20, 24, 32]),
                "umax": rng.choice([6.0, 8.0, 10.0]), "guess": rng.choice([0, 2])}
    if kind in ("train", "predict"):
        return {"kind": kind, "batch": _logint(rng, 256, 16384), "hidden": rng.choice([32, 48, 64])}
    model, precision = rng.choice([BGK, ES]), rng.choice([F64, F32])
    nv = tuple(rng.randint(10, 24) for _ in range(3))
    umax = rng.choice([6.0, 7.0, 8.0])
    rk, kn = rng.choice([SSP, LSRK]), rng.choice([1e-2, 1e-3, 2e-4])
    nu = nv[0] * nv[1] * nv[2]
    if kind == "ogrid":
        nt = _logint(rng, 8, 40)
        nv = tuple(rng.randint(16, 24) for _ in range(3))
        return _drop_name(_step("", kind, (nt, max(3, nt // 2), rng.choice([1, 2])), rng.choice([1, 2]), nv, 14.0, ES,
                                precision, rk, kn=0.01))
    if kind == "ptbox":
        n, p = rng.randint(3, 6), rng.choice([1, 2, 3])
        return _drop_name(_step("", kind, (n, n, n), p, nv, umax, model, precision, rk, kn=kn))
    p = rng.choice([1, 2, 3])
    ns = (p + 1) ** 3
    elems = math.exp(rng.uniform(math.log(2e5), math.log(4e8))) / (ns * nu)
    side = max(1.0, elems) ** (1.0 / 3.0)
    size = tuple(max(2, min(20, round(side * rng.uniform(0.8, 1.25)))) for _ in range(3))
    if kind == "box":
        delta = rng.choice([0.0, 0.0, 0.0, 2.0])
        if delta == 0.0 and rng.random() < 0.4:
            precision = DEV
        nodes = rng.choice([0, 0, 1])
        if min(nv) < 12 and delta:
            delta = 0.0
        return _drop_name(_step("", "box", size, p, nv, umax, model, precision, rk, nodes=nodes, delta=delta, kn=kn,
                                steps=rng.choice([1, 1, 2, 3]) if nu * ns * size[0] * size[1] * size[2] < 1e8 else 1))
    return _drop_name(_step("", "box", size, p, nv, umax, model, precision, rk, nodes=rng.choice([0, 1]), kn=kn,
                            kind=kind))


def _drop_name(c):
    return {k: v for k, v in c.items() if k != "name"}


# ------------------------------------------------------------------ inputs --

def _rng(seed):
    return np.random.default_rng(int(seed) + 7919)


def _grid(c):
    return workloads.grid_spec((c["n0"], c["n1"], c["n2"]), c["umax"])


def _mesh(c):
    if c["mesh"] == "box":
        return workloads.box_mesh((c["nx"], c["ny"], c["nz"]))
    if c["mesh"] == "ogrid":
        return workloads.cylinder_mesh(n_theta=c["nx"], n_r=c["ny"], n_z=c["nz"])
    return workloads.prism_tet_box_mesh(c["nx"])


def _theta_inf(c):
    return {"farfield": [1.0, 8.0 * math.sqrt(5.0 / 3.0), 0.0, 0.0, 1.0], "theta_wall": 2.0}


def _params(c):
    par = {"model": c["model"], "prandtl": (0.71 if c["model"] == ES else 1.0), "mu_ref": c["kn"] * math.sqrt(2 / math.pi),
           "theta_ref": 1.0, "omega": 0.81, "newton_tol": 1e-13, "newton_max_iter": 50, "precision": c["precision"],
           "rk": c["rk"], "guess": frdvm.GUESS_WARM if c["kind"] == "step" else frdvm.GUESS_COLD}
    if c["mesh"] == "ogrid":
        par.update(_theta_inf(c), positivity=1, prandtl=2.0 / 3.0)
    return par


def _dt(c):
    """A step of CFL number about 0.2 over (2p+1) on the thinnest element."""
    if c["mesh"] == "ogrid":
        h = 5.5 * 0.15 / (1.15 ** c["ny"] - 1.0)
        h = min(h, 0.25 / c["nz"], math.pi * 0.5 / c["nx"])
    elif c["mesh"] == "ptbox":
        h = 0.25 / c["nx"]
    else:
        h = 1.0 / max(c["nx"], c["ny"], c["nz"])
    return 0.2 * h / ((2 * c["p"] + 1) * 3.0 * c["umax"])


def _points(c, mesh):
    """Physical positions of the solution points [elements, points, 3]."""
    if c["mesh"] == "ptbox":
        return workloads.mixed_solution_points(mesh, c["p"])[:, None, :]
    xi = _points_1d(c)
    r = (xi + 1.0) / 2.0
    ref = np.stack(np.meshgrid(r, r, r, indexing="ij"), -1).transpose(2, 1, 0, 3).reshape(-1, 3)
    lo, hi = mesh["nodes"][mesh["elem_nodes"][:, 0]], mesh["nodes"][mesh["elem_nodes"][:, 7]]
    return lo[:, None, :] + ref[None] * (hi - lo)[:, None, :]


def _field(c, mesh, seed):
    """Macroscopic start [elements, points, 5]: a Taylor-Green flow with seeded smooth modes (boxes), the noisy
    Mach-8 freestream (O-grid, an impulsive start)."""
    rng = _rng(seed)
    if c["mesh"] == "ogrid":
        prim = np.tile(np.array(_theta_inf(c)["farfield"]), (mesh["n_elem"], (c["p"] + 1) ** 3, 1))
        prim[..., 0] *= 1.0 + 0.01 * rng.uniform(-1, 1, prim.shape[:2])
        return prim
    x = _points(c, mesh)
    s2 = 2 * np.pi
    U0 = 0.4
    U = [U0 * np.sin(s2 * x[..., 0]) * np.cos(s2 * x[..., 1]) * np.cos(s2 * x[..., 2]),
         -U0 * np.cos(s2 * x[..., 0]) * np.sin(s2 * x[..., 1]) * np.cos(s2 * x[..., 2]), 0 * x[..., 0]]
    rho, th = 1.0 + 0 * x[..., 0], 1.0 + 0 * x[..., 0]
    for _ in range(3):
        k = rng.integers(-1, 2, 3)
        ph = s2 * (x @ k) + rng.uniform(0, s2)
        a = rng.uniform(-0.03, 0.03, 5)
        rho = rho + a[0] * np.cos(ph)
        th = th + a[1] * np.cos(ph + 1.0)
        U = [U[d] + a[2 + d] * np.sin(ph + d) for d in range(3)]
    return np.stack([rho, U[0], U[1], U[2], th], -1)


def _axes(c, device="cuda"):
    return [torch.linspace(-c["umax"], c["umax"], n, dtype=torch.float64, device=device)
            for n in (c["n0"], c["n1"], c["n2"])]


def _sample(prim, ax, out):
    """Maxwellians of the states prim [points, 5] at every velocity node, into out [points, nodes]."""
    for s in range(0, prim.shape[0], 8192):
        q = prim[s:s + 8192]
        e = [torch.exp(-(ax[d][None, :] - q[:, 1 + d:2 + d]) ** 2 / (2 * q[:, 4:5])) for d in range(3)]
        a = (q[:, 0:1] * (2 * math.pi * q[:, 4:5]) ** -1.5)[:, :, None, None]
        g = (a * e[2][:, :, None, None]) * e[1][:, None, :, None] * e[0][:, None, None, :]
        out[s:s + 8192] = g.reshape(q.shape[0], -1).to(out.dtype)


def _state(c, mesh, seed):
    """The distribution a step starts from: Maxwellians of the macroscopic start (as the workloads'); calls that
    look at the collision alone get a mixture of two streams, out of equilibrium.  [elements, points, nodes],
    with a gas of internal energy F then G."""
    prim = torch.as_tensor(_field(c, mesh, seed), device="cuda")
    ne, ns = prim.shape[:2]
    pr = prim.reshape(-1, 5)
    nu = c["n0"] * c["n1"] * c["n2"]
    nc = 2 if c["delta"] > 0 else 1
    f = torch.empty((ne * ns, nc, nu), dtype=torch.float64 if c["precision"] == F64 else torch.float32, device="cuda")
    ax = _axes(c)
    _sample(pr, ax, f[:, 0])
    if c["kind"] != "step":
        other = pr.clone()
        other[:, 0] *= 0.5
        other[:, 1:4] += torch.tensor([0.5, -0.3, 0.2], dtype=torch.float64, device="cuda")
        other[:, 4] *= 1.3
        g = torch.empty_like(f[:, 0])
        _sample(other, ax, g)
        f[:, 0] += g
    if nc == 2:
        f[:, 1] = f[:, 0] * (0.5 * c["delta"] * 0.9)
    return f.reshape(ne, ns, nc * nu)


def _batch_states(c, seed):
    """Macroscopic states a Newton solve meets: log-normal density, bulk speed up to 0.6 u_max, log-uniform
    temperature, all well inside what the velocity grid resolves.  Moment vectors [n, 5]."""
    g = torch.Generator().manual_seed(int(seed) + 17)
    n = c["n"]
    rho = torch.exp(torch.randn(n, generator=g, dtype=torch.float64))
    d = torch.randn(n, 3, generator=g, dtype=torch.float64)
    d = d / d.norm(dim=1, keepdim=True)
    U = d * (0.6 * c["umax"] * torch.rand(n, 1, generator=g, dtype=torch.float64))
    du = 2 * c["umax"] / (c["nv"] - 1)
    lo = max(0.3, 0.9 * du * du)
    th = lo * torch.exp(torch.rand(n, generator=g, dtype=torch.float64) * math.log(max(2.0, 0.05 * c["umax"] ** 2 / lo)))
    E = 0.5 * rho * (U * U).sum(1) + 1.5 * rho * th
    return torch.cat([rho[:, None], rho[:, None] * U, E[:, None]], 1)


def _layers(H):
    return [(H, frdvm.MLP_INPUTS), (H, H), (H, H), (5, H)]


def _weights(H, seed, out_scale=1.0):
    """Network weights as the training starts from them (uniform, fan-in scaled; output affine)."""
    rng, parts = _rng(seed), []
    for m, k in _layers(H):
        lim = math.sqrt(6.0 / k)
        parts += [rng.uniform(-lim, lim, m * k), 0.05 * rng.uniform(-1, 1, m)]
    parts += [np.full(5, out_scale), np.linspace(-0.1, 0.1, 5) * out_scale]
    return np.concatenate(parts).astype(np.float32)


def _features(B, seed, H):
    g = torch.Generator().manual_seed(int(seed) + 23)
    X = torch.randn(B, frdvm.MLP_INPUTS, generator=g)
    X[:, 7:] = torch.sin(2 * math.pi * torch.rand(B, frdvm.MLP_INPUTS - 7, generator=g))
    return X, torch.randn(B, 5, generator=g)


def prepare(case, seed):
    c = case
    if c["kind"] in ("train", "predict"):
        H, B = c["hidden"], c["batch"]
        X, T = (t.cuda() for t in _features(B, seed, H))
        net = frdvm.Mlp(H)
        w = torch.as_tensor(_weights(H, seed)).cuda()
        s = {"case": c, "net": net, "w": w, "X": X, "T": T, "out": torch.empty((B, 5), device="cuda"),
             "work": net.workspace(B)}
        if c["kind"] == "train":
            s.update(m=torch.zeros_like(w), v=torch.zeros_like(w), g=torch.empty_like(w),
                     loss=torch.empty(1, device="cuda"), step=0)
        return s
    if c["kind"] == "equilibrium":
        h = frdvm.FrDvm(workloads.box_mesh(1), 1, workloads.grid_spec(c["nv"], c["umax"]),
                        {"model": BGK, "mu_ref": 1.0, "newton_tol": 1e-13, "newton_max_iter": 100})
        if c["guess"] == frdvm.GUESS_MLP:
            h.mlp_set_weights(_weights(H_NET, 5, out_scale=1e-3))
        return {"case": c, "h": h, "Q": _batch_states(c, seed).cuda().contiguous()}
    mesh = _mesh(c)
    h = frdvm.FrDvm(mesh, c["p"], _grid(c), _params(c), nodes=c["nodes"], delta=c["delta"])
    f = _state(c, mesh, seed).reshape(h.shape)
    s = {"case": c, "h": h, "f": f, "dt": _dt(c)}
    d64 = {"dtype": torch.float64, "device": "cuda"}
    if c["kind"] == "operators":
        s.update(R=torch.empty_like(f), S=torch.empty_like(f), Qp=torch.empty(h.ne * h.ns, 5, **d64))
    elif c["kind"] == "diagnostics":
        s.update(Q=torch.empty(h.ne * h.ns, 5, **d64), kn=torch.empty(h.ne * h.ns, **d64))
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "step":
        s["h"].rk_steps(s["f"], s["dt"], c["steps"])
        return s["f"]
    if c["kind"] == "operators":
        s["h"].residual(s["f"], s["R"])
        s["h"].collide(s["f"], s["S"], s["Qp"])
        return {"R": s["R"], "S": s["S"], "Qp": s["Qp"]}
    if c["kind"] == "diagnostics":
        totals = s["h"].moments(s["f"], s["Q"], totals=True)
        s["h"].kn_gll(s["f"], s["kn"])
        return {"Q": s["Q"], "totals": totals, "kn": s["kn"]}
    if c["kind"] == "equilibrium":
        z, _, _, status, _ = s["h"].equilibrium(s["Q"], c["guess"])
        return {"z": z, "status": status}
    if c["kind"] == "predict":
        return s["net"].forward(s["w"], s["X"], s["out"], s["work"])
    s["step"] += 1
    s["net"].grad(s["w"], s["X"], s["T"], s["g"], s["loss"], s["work"])
    s["net"].adam(s["w"], s["g"], s["m"], s["v"], s["step"], 1e-3)
    return {"w": s["w"], "grad": s["g"], "loss": s["loss"], "m": s["m"], "v": s["v"]}


def _points_of(c):
    """Solution points of the case's mesh."""
    n = c["p"] + 1
    if c["mesh"] == "ptbox":
        N, tet, prism = c["nx"], n * (n + 1) * (n + 2) // 6, n * n * (n + 1) // 2
        low = N // 2
        return N * N * (2 * low * prism + 6 * (N - low) * tet)
    return c["nx"] * c["ny"] * c["nz"] * n ** 3


def work(case):
    """Bytes: each input read once, each output written once.  Flops: the factorised operators (dense on
    simplices), collision and moments of every value and stage; multiply-adds of the batches."""
    c = case
    if c["kind"] in ("train", "predict"):
        H, B = c["hidden"], c["batch"]
        n = sum(m * k + m for m, k in _layers(H)) + 10
        train = c["kind"] == "train"
        return {"bytes": 4.0 * (B * 18 + (8 if train else 1) * n), "flops": (6.0 if train else 2.0) * B * n}
    if c["kind"] == "equilibrium":
        return {"bytes": c["n"] * (40 + 40 + 24.0), "flops": c["n"] * 3.0 * c["nv"] * 4 * 35}
    es = 8 if c["precision"] == F64 else 4
    nc = 2 if c["delta"] > 0 else 1
    pts = _points_of(c)
    dofs = float(pts * c["n0"] * c["n1"] * c["n2"] * nc)
    fr, coll, mom = (150 if c["mesh"] == "ptbox" else 44), 40, 8
    if c["kind"] == "operators":
        return {"bytes": 3.0 * es * dofs + 40.0 * pts, "flops": dofs * (fr + coll + mom)}
    if c["kind"] == "diagnostics":
        return {"bytes": 1.0 * es * dofs + 48.0 * pts, "flops": dofs * mom}
    return {"bytes": 2.0 * es * dofs, "flops": 3.0 * c["steps"] * dofs * (fr + coll + mom)}


# ------------------------------------------------- the same in 64 bits -------

def _points_1d(c):
    n = c["p"] + 1
    if not c["nodes"]:
        return np.polynomial.legendre.leggauss(n)[0]
    inner = np.polynomial.legendre.Legendre.basis(n - 1).deriv().roots().real
    return np.concatenate([[-1.0], np.sort(inner), [1.0]])


def _lagrange(nodes, x):
    """Values and derivatives at x of the Lagrange polynomials on nodes: [len(x), len(nodes)] each."""
    nodes, x = np.asarray(nodes, float), np.atleast_1d(np.asarray(x, float))
    n = len(nodes)
    val, der = np.ones((len(x), n)), np.zeros((len(x), n))
    for m in range(n):
        others = [j for j in range(n) if j != m]
        den = np.prod([nodes[m] - nodes[j] for j in others])
        val[:, m] = np.prod([x - nodes[j] for j in others], axis=0) / den
        der[:, m] = sum(np.prod([x - nodes[j] for j in others if j != k], axis=0) * np.ones_like(x)
                        for k in others) / den
    return val, der


class _Hexes:
    """Residual of a hexahedral mesh whose faces meet in one global frame."""

    def __init__(self, c, mesh):
        self.c, xi, n = c, _points_1d(c), c["p"] + 1
        self.n, self.ns, self.ne = n, n ** 3, mesh["n_elem"]
        dev = {"dtype": torch.float64, "device": "cuda"}
        lam = np.concatenate([_lagrange(xi, [-1.0])[0], _lagrange(xi, [1.0])[0]])
        xg, wg = np.polynomial.legendre.leggauss(n + 1)
        L = _lagrange(xi, xg)[0]
        mass = L.T @ (wg[:, None] * L)
        self.D = torch.as_tensor(_lagrange(xi, xi)[1], **dev)
        self.lam = torch.as_tensor(lam, **dev)
        self.lift = torch.as_tensor(np.linalg.solve(mass, lam.T).T, **dev)  # [side, point]
        self.w1 = mass.sum(1)
        # geometry: cofactors |J| grad xi_d at the points, outward area normals at the face points
        g = np.array([-1.0, 1.0]) if mesh["geom_order"] == 1 else np.array([-1.0, 0.0, 1.0])
        X = mesh["nodes"][mesh["elem_nodes"]]  # [e, geometry nodes, 3]

        def cofactors(x, y, z):
            (lx, dx), (ly, dy), (lz, dz) = (_lagrange(g, t) for t in (x, y, z))
            shape = [np.einsum("pk,pj,pi->pkji", *t).reshape(len(x), -1)
                     for t in ((lz, ly, dx), (lz, dy, lx), (dz, ly, lx))]
            t = [np.einsum("pa,eac->epc", s, X) for s in shape]  # dx/dxi_d
            a = [np.cross(t[1], t[2]), np.cross(t[2], t[0]), np.cross(t[0], t[1])]
            return np.stack(a, 2), np.einsum("epc,epc->ep", t[0], a[0])

        k, j, i = (t.reshape(-1) for t in np.meshgrid(xi, xi, xi, indexing="ij"))
        S, J = cofactors(i, j, k)
        b, a = (t.reshape(-1) for t in np.meshgrid(xi, xi, indexing="ij"))
        one = np.ones_like(a)
        nrm = []
        for face in range(6):
            d, sgn = face // 2, 2.0 * (face % 2) - 1.0
            pos = [sgn * one, a, b] if d == 0 else [a, sgn * one, b] if d == 1 else [a, b, sgn * one]
            nrm.append(sgn * cofactors(*pos)[0][:, :, d])
        self.S, self.J = torch.as_tensor(S, **dev), torch.as_tensor(J, **dev)
        self.nrm = torch.as_tensor(np.stack(nrm, 1), **dev)  # [e, 6, face point, 3]
        w = self.w1
        self.W = torch.as_tensor(np.einsum("k,j,i->kji", w, w, w).reshape(-1)[None] * J, **dev)
        self.nb = torch.as_tensor(mesh["nbr_elem"].astype(np.int64), device="cuda")
        self.nf = torch.as_tensor(mesh["nbr_face"].astype(np.int64), device="cuda")
        self.bc = torch.as_tensor(mesh["bc"].astype(np.int64), device="cuda")

    def traces(self, f):
        """f [e, point, k] at the points of the six faces: [e, 6, face point, k]."""
        n = self.n
        v = f.reshape(self.ne, n, n, n, -1)
        out = torch.empty(self.ne, 6, n * n, f.shape[-1], dtype=f.dtype, device=f.device)
        for face in range(6):
            d, lam = face // 2, self.lam[face % 2]
            line = [v.select(3 - d, m) for m in range(n)]
            out[:, face] = sum(lam[m] * line[m] for m in range(n)).reshape(self.ne, n * n, -1)
        return out

    def chunks(self, nk):
        step = max(64, int(1.5e8 / (self.ne * self.ns)))
        return [slice(s, min(nk, s + step)) for s in range(0, nk, step)]

    def residual(self, f, V):
        """f [e, point, component x node] at velocities V [node, 3]."""
        R = torch.empty_like(f)
        nu, n = V.shape[0], self.n
        wall = (self.nb < 0) & (self.bc == 2)
        far = (self.nb < 0) & (self.bc == 1)
        if wall.any():
            we, wf = wall.nonzero(as_tuple=True)
            nw = self.nrm[we, wf]
            th = _theta_inf(self.c)["theta_wall"]
            mw = (2 * math.pi * th) ** -1.5 * torch.exp(-(V * V).sum(1) / (2 * th))
            q = _theta_inf(self.c)["farfield"]
            U = torch.tensor(q[1:4], dtype=V.dtype, device=V.device)
            finf = q[0] * (2 * math.pi * q[4]) ** -1.5 * torch.exp(-((V - U) ** 2).sum(1) / (2 * q[4]))
            wq = _weights3(self.c)
            out = torch.zeros(nw.shape[:2], dtype=f.dtype, device=f.device)
            inn = torch.zeros_like(out)
            for ks in self.chunks(nu):
                un = nw @ V[ks].T
                line = f.reshape(self.ne, n, n, n, -1)[we][..., ks]  # wall faces are faces 0
                t = sum(self.lam[0][m] * line[:, :, :, m] for m in range(n)).reshape(len(we), n * n, -1)
                out += (wq[ks] * un.clamp(min=0) * t).sum(-1)
                inn += (wq[ks] * (-un).clamp(min=0) * mw[ks]).sum(-1)
            rw = out / inn
        nb, nf = self.nb.clamp(min=0), self.nf.long()
        for comp in range(f.shape[-1] // nu):
            for ks in self.chunks(nu):
                kf = slice(comp * nu + ks.start, comp * nu + ks.stop)
                v, u = f[:, :, kf].contiguous(), V[ks].T.contiguous()
                tr = self.traces(v)
                r = torch.zeros_like(v).reshape(self.ne, n, n, n, -1)
                for d in range(3):
                    F = ((self.S[:, :, d] @ u) * v).reshape(self.ne, n, n, n, -1)
                    for i in range(n):
                        r.select(3 - d, i).add_(sum(self.D[i, m] * F.select(3 - d, m) for m in range(n)))
                    for side in range(2):
                        face = 2 * d + side
                        un = self.nrm[:, face] @ u
                        ext = tr[nb[:, face], nf[:, face]]
                        if wall.any():
                            sel = wf == face
                            ext[we[sel]] = rw[sel][..., None] * mw[ks]
                            ext[far[:, face]] = finf[ks]
                        jump = (un.clamp(max=0) * (ext - tr[:, face])).reshape(self.ne, n, n, -1)
                        for i in range(n):
                            r.select(3 - d, i).add_(self.lift[side, i] * jump)
                R[:, :, kf] = -r.reshape(v.shape) / self.J[..., None]
        return R

    def limit(self, f):
        """Positivity: every value's element polynomial scaled about its mean until its least point and face
        value is zero."""
        for ks in self.chunks(f.shape[-1]):
            v = f[:, :, ks]
            mean = (v * self.W[..., None]).sum(1, keepdim=True) / self.W.sum(1)[:, None, None]
            low = torch.minimum(v.amin(1, keepdim=True), self.traces(v.contiguous()).flatten(1, 2).amin(1, keepdim=True))
            th = torch.where(low < 0, torch.where(mean > 0, mean / (mean - low), torch.zeros_like(mean)),
                             torch.ones_like(mean))
            f[:, :, ks] = mean + th * (v - mean)


class _Simplices:
    """Residual of a prism / tetrahedron mesh (straight elements, nodal operators with exact mass matrices)."""

    def __init__(self, c, mesh):
        p, dev = c["p"], {"dtype": torch.float64, "device": "cuda"}
        verts = {1: [[-1, -1, -1], [1, -1, -1], [-1, 1, -1], [-1, -1, 1], [1, -1, 1], [-1, 1, 1]],
                 2: [[-1, -1, -1], [1, -1, -1], [-1, 1, -1], [-1, -1, 1]]}
        g, w = np.polynomial.legendre.leggauss(p + 4)
        g, w = 0.5 * (g + 1), 0.5 * w
        N, et = mesh["N"], mesh["elem_type"]
        off = np.concatenate([[0], np.cumsum([{1: (p + 1) ** 2 * (p + 2) // 2, 2: (p + 1) * (p + 2) * (p + 3) // 6}[int(t)]
                                              for t in et])])
        xyz = workloads.mixed_solution_points(mesh, p)
        owner = np.repeat(np.arange(len(et)), np.diff(off))

        def key(e, x):  # (element, position modulo the period) as one integer
            q = np.round((x % 1.0) * 20011.0).astype(np.int64) % 20011
            return ((e.astype(np.int64) * 20011 + q[:, 0]) * 20011 + q[:, 1]) * 20011 + q[:, 2]

        keys = key(owner, xyz)
        order = np.argsort(keys)
        self.types = []
        for t in (1, 2):
            el = np.nonzero(et == t)[0]
            if not len(el):
                continue
            ref, rv = workloads.mixed_reference_points(t, p), np.array(verts[t], float)
            ns = len(ref)
            ex = [(a, b, k) for k in range(p + 1) for b in range(p + 1) for a in range(p + 1)
                  if (a + b <= p if t == 1 else a + b + k <= p)]

            def mono(x, d=-1):
                cols = []
                for e3 in ex:
                    q, co = list(e3), 1.0
                    if d >= 0:
                        co, q[d] = float(q[d]), max(q[d] - 1, 0)
                    cols.append(co * x[:, 0] ** q[0] * x[:, 1] ** q[1] * x[:, 2] ** q[2])
                return np.stack(cols, 1)

            C = np.linalg.inv(mono(ref))
            pts, wts = [], []
            for i in range(len(g)):
                for j in range(len(g)):
                    for k in range(len(g)):
                        a, b = g[i], g[j] * (1 - g[i])
                        if t == 1:
                            pts.append([2 * a - 1, 2 * b - 1, 2 * g[k] - 1])
                            wts.append(8 * w[i] * w[j] * w[k] * (1 - g[i]))
                        else:
                            pts.append([2 * a - 1, 2 * b - 1, 2 * g[k] * (1 - a - b) - 1])
                            wts.append(8 * w[i] * w[j] * w[k] * (1 - g[i]) * (1 - a - b))
            Lq = mono(np.array(pts)) @ C
            mass = Lq.T @ (np.array(wts)[:, None] * Lq)
            X = mesh["nodes"][mesh["elem_nodes"][el][:, :len(rv)]]
            ax = [1, 2, 3]
            A = np.stack([X[:, a] - X[:, 0] for a in ax], 2) / 2.0  # dx/dxi
            Ai, J = np.linalg.inv(A), np.linalg.det(A)
            own = off[el][:, None] + np.arange(ns)
            faces = []
            for f, fv in enumerate(workloads.MIXED_FACE_VERTS[t]):
                P = rv[fv]
                e1, e2 = P[1] - P[0], (P[2] if len(fv) == 3 else P[3]) - P[0]
                nref = np.cross(e1, e2)
                on = np.nonzero(np.abs((ref - P[0]) @ nref) < 1e-9)[0]
                fp, fw = [], []
                for i in range(len(g)):
                    for j in range(len(g)):
                        v = g[j] * ((1 - g[i]) if len(fv) == 3 else 1.0)
                        fp.append(P[0] + g[i] * e1 + v * e2)
                        fw.append(w[i] * w[j] * ((1 - g[i]) if len(fv) == 3 else 1.0))
                Lf = mono(np.array(fp)) @ C
                lift = np.linalg.solve(mass, Lf.T @ (np.array(fw)[:, None] * Lf))[:, on]  # unit parameter area
                E1, E2 = A @ e1, A @ e2
                an = np.cross(E1, E2)  # area vector of the parameter square
                out = X.mean(1) - X[:, fv].mean(1)
                an = an * -np.sign((an * out).sum(1))[:, None]
                m = np.repeat(mesh["nbr_elem"][el, f], len(on))
                at = np.searchsorted(keys[order], key(m, xyz[own[:, on]].reshape(-1, 3)))
                nbp = order[at].reshape(len(el), len(on))
                faces.append((torch.as_tensor(on, device="cuda"), torch.as_tensor(lift, **dev),
                              torch.as_tensor(an / J[:, None], **dev), torch.as_tensor(nbp, device="cuda")))
            D = torch.as_tensor(np.stack([mono(ref, d) @ C for d in range(3)]), **dev)
            self.types.append((torch.as_tensor(own, device="cuda"), D, torch.as_tensor(Ai, **dev), faces))

    def residual(self, f, V):
        R = torch.empty_like(f)
        v0, r0 = f.reshape(f.shape[0], -1), R.reshape(f.shape[0], -1)
        step = max(64, int(1.5e8 / f.shape[0]))
        for s in range(0, V.shape[0], step):
            v, u = v0[:, s:s + step].contiguous(), V[s:s + step].T.contiguous()
            for own, D, Ai, faces in self.types:
                x = v[own]
                r = torch.zeros_like(x)
                for a in range(3):
                    r -= (Ai[:, a] @ u)[:, None] * torch.matmul(D[a], x)
                for on, lift, an, nbp in faces:
                    jump = (an @ u).clamp(max=0)[:, None] * (v[nbp] - x[:, on])
                    r -= torch.matmul(lift, jump)
                r0[own.reshape(-1), s:s + step] = r.reshape(-1, r.shape[-1])
        return R

    def limit(self, f):
        pass


def _weights3(c):
    """Trapezoid weights of the velocity nodes."""
    one = []
    for x in _axes(c):
        w = torch.full_like(x, float(x[1] - x[0]))
        w[0] *= 0.5
        w[-1] *= 0.5
        one.append(w)
    return (one[2][:, None, None] * one[1][None, :, None] * one[0][None, None, :]).reshape(-1)


def _nodes3(c):
    ax = _axes(c)
    z, y, x = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    return torch.stack([x, y, z], -1).reshape(-1, 3)


_PAIRS = [(0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)]


def _quartics():
    """Monomials of degree <= 4 and, for the ten of degree <= 2 (1, x, y, z, xx, yy, zz, xy, xz, yz), where the
    product of each two stands among them."""
    e2 = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1)]
    e2 += [tuple((a == d) + (b == d) for d in range(3)) for a, b in _PAIRS]
    e4 = sorted({tuple(x + y for x, y in zip(a, b)) for a in e2 for b in e2})
    at = [[e4.index(tuple(x + y for x, y in zip(a, b))) for b in e2] for a in e2]
    return e2, e4, torch.tensor(at, device="cuda")


def _monomials(v, exps):
    return torch.stack([v[:, 0] ** a * v[:, 1] ** b * v[:, 2] ** c for a, b, c in exps], 0)


def _rows(V, s, B):
    """In the frame c = (v - V) / s: the rows 1, c, |c|^2 / 2 and 1, c, -q / 2 with q = (v-V)^T B (v-V) as
    combinations of the ten monomials of v, [points, 5, 10] each."""
    n = V.shape[0]
    P = torch.zeros(n, 5, 10, dtype=V.dtype, device=V.device)
    P[:, 0, 0] = 1
    for d in range(3):
        P[:, 1 + d, 1 + d] = 1 / s
        P[:, 1 + d, 0] = -V[:, d] / s
    Q = P.clone()
    P[:, 4, 0] = 0.5 * (V * V).sum(1) / s ** 2
    for d in range(3):
        P[:, 4, 1 + d] = -V[:, d] / s ** 2
        P[:, 4, 4 + d] = 0.5 / s ** 2
    BV = (B @ V[:, :, None])[:, :, 0]
    Q[:, 4, 0] = -0.5 * (V * BV).sum(1)
    for d in range(3):
        Q[:, 4, 1 + d] = BV[:, d]
    for m, (a, b) in enumerate(_PAIRS):
        Q[:, 4, 4 + m] = -0.5 * B[:, a, b] if a == b else -B[:, a, b]
    return P, Q


class _Gas:
    """Moments, conservative equilibria and relaxation of points [points, component x node]."""

    def __init__(self, c, V, w, shift, model, prandtl, mu_ref, delta):
        self.V, self.w, self.model, self.Pr, self.mu, self.delta = V, w, model, prandtl, mu_ref, delta
        e2, e4, self.at = _quartics()
        v = V - shift
        self.m2, self.m4 = _monomials(v, e2), _monomials(v, e4)
        self.shift = shift
        self.step = max(256, int(6e7 / V.shape[0]))

    def equilibrium(self, rho, U, Pi, th):
        """z of exp(z0 + z.c - z4 q / 2) (frame of U and theta) with the moments of the state, and the monomial
        coefficients of its exponent for g."""
        n = rho.shape[0]
        eye = torch.eye(3, dtype=rho.dtype, device=rho.device)
        if self.model == ES:
            T = (th / self.Pr)[:, None, None] * eye + (1 - 1 / self.Pr) * Pi / rho[:, None, None]
        else:
            T = th[:, None, None] * eye
        B = torch.linalg.inv(T)
        s = th.sqrt()
        P, F = _rows(U - self.shift, s, B)
        z = torch.zeros(n, 5, dtype=rho.dtype, device=rho.device)
        z[:, 0] = -1.5 * math.log(2 * math.pi) + 0.5 * torch.logdet(B * th[:, None, None])
        z[:, 4] = 1
        target = torch.tensor([1, 0, 0, 0, 1.5], dtype=rho.dtype, device=rho.device)
        wm = (self.w * self.m4).T.contiguous()

        def sums(zz, i):
            out = []
            for a in range(0, len(i), self.step):
                j = i[a:a + self.step]
                ex = (zz[a:a + self.step, None] @ F[j])[:, 0] @ self.m2
                out.append((torch.exp(ex) @ wm) * th[j, None] ** -1.5)
            H = torch.cat(out)[:, self.at]
            r = (P[i] @ H[:, :, :1])[:, :, 0] - target
            return r, P[i] @ H @ F[i].transpose(1, 2)

        todo = torch.arange(n, device=rho.device)
        r, J = sums(z, todo)
        for _ in range(40):
            dz = -torch.linalg.solve(J, r)
            a = torch.ones(len(todo), 1, dtype=z.dtype, device=z.device)
            for _ in range(8):
                zt = z[todo] + a * dz
                zt[:, 4] = zt[:, 4].clamp(min=1e-3)
                rt, Jt = sums(zt, todo)
                worse = ~(rt.norm(dim=1) <= r.norm(dim=1)) & (r.norm(dim=1) > 1e-10)
                if not worse.any():
                    break
                a[worse] *= 0.5
            z[todo] = zt
            keep = ~(rt.abs().amax(1) < 1e-12) & (dz.abs().amax(1) > 1e-13)
            todo, r, J = todo[keep], rt[keep], Jt[keep]
            if not len(todo):
                break
        coef = (z[:, None] @ F)[:, 0]
        coef[:, 0] += torch.log(rho) - 1.5 * torch.log(th)
        return z, coef, B

    def state(self, f):
        """rho, U, pressure tensor, theta and the integral of G."""
        nu = self.V.shape[0]
        m = torch.cat([f[a:a + 4 * self.step, :nu].double() @ (self.w * self.m2).T
                       for a in range(0, f.shape[0], 4 * self.step)])
        rho, V = m[:, 0], m[:, 1:4] / m[:, 0:1]
        Pi = torch.empty(len(rho), 3, 3, dtype=m.dtype, device=m.device)
        for k, (a, b) in enumerate(_PAIRS):
            Pi[:, a, b] = Pi[:, b, a] = m[:, 4 + k] - rho * V[:, a] * V[:, b]
        G = f[:, nu:].double() @ self.w if f.shape[1] > nu else torch.zeros_like(rho)
        th = (Pi.diagonal(dim1=1, dim2=2).sum(1) + 2 * G) / ((3 + self.delta) * rho)
        return rho, V + self.shift, Pi, th, G

    def source(self, f, into):
        """into += (g - f) / tau; returns the primitive state of g."""
        rho, U, Pi, th, _ = self.state(f)
        z, coef, B = self.equilibrium(rho, U, Pi, th)
        pr = self.Pr if self.model == ES else 1.0
        itau = pr * rho * th / (self.mu * th ** 0.81)
        nu = self.V.shape[0]
        for a in range(0, f.shape[0], self.step):
            s = slice(a, a + self.step)
            g = torch.exp(coef[s] @ self.m2)
            into[s, :nu] += (g - f[s, :nu]) * itau[s, None]
            if f.shape[1] > nu:
                into[s, nu:] += (0.5 * self.delta * th[s, None] * g - f[s, nu:]) * itau[s, None]
        A = B * th[:, None, None]
        m = torch.linalg.solve(A, z[:, 1:4]) / z[:, 4:5]
        mAm = (m[:, None] @ A @ m[:, :, None])[:, 0, 0]
        rp = rho * torch.exp(z[:, 0] + 0.5 * z[:, 4] * mAm) * (2 * math.pi / z[:, 4]) ** 1.5 / torch.linalg.det(A).sqrt()
        return torch.cat([rp[:, None], U + th.sqrt()[:, None] * m, (th / z[:, 4])[:, None]], 1)


def _exact_net(c, seed):
    H, B = c["hidden"], c["batch"]
    X, T = (t.cuda().double() for t in _features(B, seed, H))
    w = torch.as_tensor(_weights(H, seed)).cuda().double().requires_grad_(True)
    a, o = X, 0
    for layer, (m, k) in enumerate(_layers(H)):
        a = a @ w[o:o + m * k].reshape(m, k).T + w[o + m * k:o + m * k + m]
        o += m * k + m
        if layer < 3:
            a = a * torch.sigmoid(a)
    if c["kind"] == "predict":
        return (a * w[o:o + 5] + w[o + 5:o + 10]).detach()
    loss = 0.5 * ((a - T) ** 2).sum() / B
    loss.backward()
    g = w.grad.clone()
    g[o:] = 0
    w = w.detach()
    m1, m2 = 0.1 * g, 0.001 * g * g
    step = 1e-3 * (m1 / (1 - 0.9)) / ((m2 / (1 - 0.999)).sqrt() + 1e-8)
    return {"w": w - step, "grad": g, "loss": loss.detach().reshape(1), "m": m1, "v": m2}


def exact(case, seed):
    c = case
    with torch.no_grad() if c["kind"] != "train" else torch.enable_grad():
        if c["kind"] in ("train", "predict"):
            return _exact_net(c, seed)
        if c["kind"] == "equilibrium":
            Q = _batch_states(c, seed).cuda()
            k = dict(c, n0=c["nv"], n1=c["nv"], n2=c["nv"])
            V, w = _nodes3(k), _weights3(k)
            gas = _Gas(k, V, w, torch.zeros(3, dtype=V.dtype, device="cuda"), BGK, 1.0, 1.0, 0.0)
            rho, U = Q[:, 0], Q[:, 1:4] / Q[:, :1]
            th = (2 / 3) * (Q[:, 4] / rho - 0.5 * (U * U).sum(1))
            if c["n"] * V.shape[0] > 8e9:
                return None
            return {"z": gas.equilibrium(rho, U, None, th)[0], "status": None}
        mesh = _mesh(c)
        f = _state(c, mesh, seed).double()
        V, w = _nodes3(c), _weights3(c)
        par = _params(c)
        shift = torch.tensor(par["farfield"][1:4] if c["mesh"] == "ogrid" else [0.0, 0.0, 0.0],
                             dtype=V.dtype, device="cuda")
        gas = _Gas(c, V, w, shift, c["model"], par["prandtl"], par["mu_ref"], c["delta"])
        fr = _Simplices(c, mesh) if c["mesh"] == "ptbox" else _Hexes(c, mesh)
        flat = (f.shape[0] * f.shape[1], f.shape[2])
        if c["kind"] == "operators":
            S = torch.zeros_like(f)
            Qp = gas.source(f.reshape(flat), S.reshape(flat))
            return {"R": fr.residual(f, V), "S": S, "Qp": Qp}
        if c["kind"] == "diagnostics":
            rho, U, Pi, th, G = gas.state(f.reshape(flat))
            E = 0.5 * (Pi.diagonal(dim1=1, dim2=2).sum(1) + rho * (U * U).sum(1)) + G
            Q = torch.cat([rho[:, None], rho[:, None] * U, E[:, None]], 1)
            n = c["p"] + 1
            r = rho.reshape(f.shape[0], n, n, n)
            dr = [torch.einsum(eq, fr.D, r)
                  for eq in ("im,eljm->elji", "im,elmj->elij", "im,emlj->eilj")]
            g2 = sum((2 * h * d) ** 2 for h, d in zip((c["nx"], c["ny"], c["nz"]), dr)).reshape(-1)
            lam = par["mu_ref"] * th ** 0.81 / rho * torch.sqrt(math.pi / (2 * th))
            return {"Q": Q, "totals": (fr.W.reshape(-1, 1) * Q).sum(0), "kn": lam * g2.sqrt() / rho}
        dt, dF, f0 = _dt(c), None, None
        for stage in range(3 * c["steps"]):
            st = stage % 3
            L = fr.residual(f, V)
            gas.source(f.reshape(flat), L.reshape(flat))
            if c["rk"] == SSP:
                f0 = f.clone() if st == 0 else f0
                b = (1.0, 0.25, 2.0 / 3.0)[st]
                f.add_(L, alpha=dt).mul_(b)
                if st:
                    f.add_(f0, alpha=(0.0, 0.75, 1.0 / 3.0)[st])
            else:
                L.mul_(dt)
                dF = L if st == 0 else dF.mul_((0.0, -5.0 / 9.0, -153.0 / 128.0)[st]).add_(L)
                f.add_(dF, alpha=(1.0 / 3.0, 15.0 / 16.0, 8.0 / 15.0)[st])
            if par.get("positivity"):
                fr.limit(f)
        return f

"""General meshes store a trace row only where a velocity of the wave leaves
within a margin; a specular face reads its own row at the mirrored velocity.
The margins that set-up puts beside the normals, in the kernels' store and
read rules (applied here in numpy): no velocity of a specular face may read a
row that no wave stores, at every tilt of the plane that set-up accepts (the
normal's axis component equal to its length to 1e-12, up to 1.4e-6 rad), in
every axis, on grids with and without a node of zero velocity."""
import json

import pytest

from hipstub import run

CODE = """
import json
def unstored(n4, grid, ax, real):
    # n4: normals and margins [points][4] of one face; a row is stored per 64 velocities
    a = [np.linspace(grid["umin"][d], grid["umax"][d], grid["n"][d]) for d in range(3)]
    n = grid["n"]
    iv = np.stack(np.meshgrid(*[np.arange(m) for m in n], indexing="ij"), -1).transpose(2, 1, 0, 3).reshape(-1, 3)
    u = np.stack([a[d][iv[:, d]] for d in range(3)], -1).astype(real)
    st = (1, n[0], n[0] * n[1])[ax]
    k = np.arange(len(u))
    km = k + (n[ax] - 1 - 2 * iv[:, ax]) * st
    bad = 0
    for r in n4.astype(real):
        un = r[0] * u[:, 0] + r[1] * u[:, 1] + r[2] * u[:, 2]
        keep = un + r[3] * np.abs(u).sum(1) > 0
        wave = np.add.reduceat(keep.astype(int), np.arange(0, len(u), 64)) > 0
        bad += int((~wave[km[un < 0] // 64]).sum())
    return bad

base = W.box_mesh((1, 1, 2), periodic=False)
out, seen = [], 0
for ax in range(3):
    for to in range(3):
        if to == ax: continue
        for tilt in (0.0, 1e-9, 3e-8, -1e-7, 1e-6, -1.4e-6):
            mesh = dict(base, nodes=base["nodes"].copy(), bc=base["bc"].copy())
            mesh["nodes"][:, ax] += tilt * mesh["nodes"][:, to]   # the faces of axis ax tilt towards axis `to`
            for f in (2 * ax, 2 * ax + 1):
                mesh["bc"][:, f] = np.where(mesh["nbr_elem"][:, f] < 0, 3, 0)
            for n in ((20, 21, 20), (24, 24, 25), (21, 20, 20), (7, 5, 3), (64, 2, 3), (8, 8, 8)):
                grid = W.grid_spec(n, 5.0)
                h = F.FrDvm(mesh, 2, grid)
                pts = 2 * 6 * 9
                for real, size in ((np.float64, 8), (np.float32, 4)):
                    tab = (C.c_double if size == 8 else C.c_float) * (pts * 4)
                    # the table with the margins behind a face's normals, and the one with each at its normal
                    p, q = hip.stub_find(pts * 4 * size, 0), hip.stub_find(pts * 4 * size, 1)
                    assert p and q and not hip.stub_find(pts * 4 * size, 2)
                    a, b = (np.array(tab.from_address(x)).reshape(2, 6, 36) for x in (p, q))
                    if not np.array_equal(a[..., 27:], b.reshape(2, 6, 9, 4)[..., 3]): a, b = b, a
                    n4 = b.reshape(2, 6, 9, 4)
                    assert np.array_equal(a[..., 27:], n4[..., 3]) and np.array_equal(a[..., :27].reshape(2, 6, 9, 3), n4[..., :3])
                    for e in range(2):
                        for f in (2 * ax, 2 * ax + 1):
                            if mesh["bc"][e, f] != 3: continue
                            seen += 1
                            b = unstored(n4[e, f], grid, ax, real)
                            if b: out.append([ax, to, tilt, n, size, b])
                h.destroy()
print(json.dumps([seen, out]))
"""


def test_mirrored_rows_are_stored(tmp_path):
    seen, bad = json.loads(run(tmp_path, CODE).splitlines()[-1])
    assert seen > 1000
    assert not bad, bad[:8]

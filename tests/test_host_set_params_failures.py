"""fr_dvm_set_params when a device allocation fails, at each of its
allocations in turn, on handles of every mesh family that already work under
other parameters: the call says so, every compute entry point then refuses
without a launch, the same call made again succeeds and leaves the buffers of
a handle that never failed, and so do the earlier parameters; destroying the
handle returns all memory."""
import json

import pytest

from hipstub import run

CODE = """
import json
def params(**kw):
    p = F._Params()
    F.lib().fr_dvm_default_params(C.byref(p))
    for k, v in dict(mu_ref=0.02, prandtl=0.71, **kw).items(): setattr(p, k, v)
    return p
L = F.lib()
def calls(h):
    x = C.c_void_p(4096)  # (a device pointer: never read by the stand-in)
    return [L.fr_dvm_moments(h._h, x, x, None), L.fr_dvm_residual(h._h, x, C.c_void_p(8192)),
            L.fr_dvm_collide(h._h, x, C.c_void_p(8192), None, 0), L.fr_dvm_rk_steps(h._h, x, 1e-3, 1),
            L.fr_dvm_equilibrium(h._h, x, 8, 0, x, x, x, x, x)]
grid = W.grid_spec((9, 8, 7), 5.0)
box = W.box_mesh((3, 2, 2))
bgk, es = dict(model=0), dict(model=1)
CASES = {
    "box bgk -> es": (box, 3, {}, bgk, es),
    "box fp64 -> dev": (box, 3, {}, es, dict(es, precision=2)),
    "box -> limiter": (box, 2, {}, es, dict(es, positivity=1)),
    "box pair -> limiter": (box, 2, dict(delta=2.0), es, dict(es, positivity=1)),
    "gll fp64 -> fp32 low storage": (box, 3, dict(nodes=1), bgk, dict(es, precision=1, rk=1)),
    "mixed": (W.prism_tet_box_mesh(3), 2, {}, bgk, dict(es, precision=1, rk=1)),
    "general": (W.cylinder_mesh(4, 2, 1), 2, {}, bgk, dict(es, precision=1)),
}
mesh, p, kw, A, B = CASES[CASE]
base = hip.stub_live()
def handle(*sets):
    h = F.FrDvm(mesh, p, grid, **kw)
    for s in sets:
        rc = L.fr_dvm_set_params(h._h, C.byref(params(**s)))
        assert rc == 0, (rc, h.last_error(), s)
    return h
h = handle(A); hip.stub_fail_at(-1)
assert L.fr_dvm_set_params(h._h, C.byref(params(**B))) == 0
n = hip.stub_allocs()
want = hip.stub_live()
assert all(rc == 0 for rc in calls(h)), h.last_error()
h.destroy()
assert hip.stub_live() == base, "leak"
bad = []
for k in range(n):
    for again in (B, A):
        h = handle(A)
        hip.stub_fail_at(k)
        rc = L.fr_dvm_set_params(h._h, C.byref(params(**B)))
        hip.stub_fail_at(-1)
        if rc != -2: bad.append(("not refused", k, rc))
        l0 = hip.stub_launches()
        r = calls(h)
        if any(x != -1 for x in r) or hip.stub_launches() != l0: bad.append(("ran", k, r))
        rc = L.fr_dvm_set_params(h._h, C.byref(params(**again)))
        if rc or (again is B and hip.stub_live() != want): bad.append(("again", k, rc, hip.stub_live(), want))
        if any(calls(h)): bad.append(("after", k))
        h.destroy()
        if hip.stub_live() != base: bad.append(("leak", k)); base = hip.stub_live()
print(json.dumps([n, bad]))
"""


@pytest.mark.parametrize("case", ["box bgk -> es", "box fp64 -> dev", "box -> limiter", "box pair -> limiter",
                                  "gll fp64 -> fp32 low storage", "mixed", "general"])
def test_a_failed_allocation_leaves_a_handle_that_refuses(tmp_path, case):
    n, bad = json.loads(run(tmp_path, f"CASE = {case!r}\n" + CODE).splitlines()[-1])
    print(case, n, "allocations")
    assert not bad, (n, bad[:10])

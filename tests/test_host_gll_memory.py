"""Gauss-Lobatto boxes hold a stage value in place of two buffers of traces.
At every order, storage form and scheme, on velocity grids with and without
nodes of zero velocity, such a handle owns no more device memory than the same
box on Gauss points (which keeps traces), so that what fits beside the one
fits beside the other; and a change of scheme allocates nothing."""
import json

import pytest

from hipstub import run

CODE = """
import json
out, no_traces = [], 0
def g(n, umax):
    umin = [-u if m > 1 else 0.0 for m, u in zip(n, umax)]
    return {"n": list(n), "umin": umin, "umax": [float(u) if m > 1 else 0.0 for m, u in zip(n, umax)]}
mesh = W.box_mesh((3, 2, 2))
for n in ((8, 8, 8), (9, 8, 7), (9, 9, 9), (3, 3, 3), (16, 16, 16), (9, 1, 1), (8, 3, 1), (64, 1, 64), (1, 1, 1)):
    for p in (1, 2, 3):
        for prec in (0, 1, 2):
            for delta in (0.0, 2.0):
                if prec == 2 and delta: continue
                for rk in (0, 1):
                    own = []
                    for nodes in (0, 1):
                        h = F.FrDvm(mesh, p, g(n, (5.0, 4.0, 6.0)), dict(model=1, prandtl=0.7, mu_ref=0.1, precision=prec, rk=rk),
                                    nodes=nodes, delta=delta)
                        own.append(h.sizes()["workspace_bytes"])
                        live = hip.stub_live()
                        h.set_params(model=1, prandtl=0.7, mu_ref=0.1, precision=prec, rk=1 - rk)
                        if hip.stub_live() != live: out.append(["scheme change", n, p, prec, rk, nodes])
                        h.destroy()
                    if own[1] > own[0]: out.append(["memory", n, p, prec, delta, rk, own])
                    no_traces += own[1] < own[0]
print(json.dumps([no_traces, out]))
"""


def test_gll_boxes_own_no_more_than_gauss_boxes(tmp_path):
    less, bad = json.loads(run(tmp_path, CODE).splitlines()[-1])
    assert not bad, bad[:8]
    assert less > 100

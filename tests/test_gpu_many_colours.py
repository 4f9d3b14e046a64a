"""Meshes of five and more colours: the cells of a colour split further, which is a colouring too and leaves the order
of the relaxations, so the results stay those of the oracle's sweeps.  Up to 16 colours run in one workgroup or in blocks
(windows of a period's divisors, for 13 and 16 colours eight of them), more of them as a launch per colour."""
import numpy as np
import pytest

import oracle
from paper_2303_10846_amd.cases import configs

pytestmark = pytest.mark.gpu

TOL = 1e-11  # the FP64 parity bar of the suite


def rel(a, b):
    return float(np.max(np.abs(a - b)) / max(float(np.max(np.abs(b))), 1e-300))


def split_colours(mesh, m):
    off = [int(x) for x in mesh["color_offsets"]]
    while len(off) - 1 < m:
        k = max(range(len(off) - 1), key=lambda c: off[c + 1] - off[c])
        off.insert(k + 1, (off[k] + off[k + 1]) // 2)
    return dict(mesh, color_offsets=np.array(off, dtype=np.int64))


@pytest.mark.parametrize("kind,n,colours,n_macro,form", [
    ("tet", 2, 5, 3, "workgroup"), ("hex", 3, 16, 2, "workgroup"), ("hex", 3, 17, 2, "colours"),
    ("hex", 6, 5, 3, "blocks"), ("tet", 6, 8, 2, "blocks"), ("tet", 6, 13, 2, "blocks"), ("hex", 10, 16, 2, "blocks"),
    ("mixed", 5, 7, 3, "blocks"), ("tet", 6, 17, 2, "colours"), ("tet", 12, 11, 2, "blocks"),
    ("tet", 20, 16, 1, "wide blocks"),  # windows of 2 steps: the seventh of the eight
])
def test_macro_sweeps_of_many_colours(kind, n, colours, n_macro, form):
    from paper_2303_10846_amd.binding import Solver
    c = configs.open_box_case(n=n, nv_side=3, kind=kind)
    c["mesh"] = split_colours(c["mesh"], colours)
    num = dict(c["num"], n_macro=n_macro, n_micro=1)
    o = oracle.Oracle(c, num=num)
    o.init_equilibrium(c["W0"])
    o.iterate(2)
    s = Solver(c, precision="fp64", num=num)
    s.set_state(*o.get_state())
    for k in range(2):
        s.iterate(1)
        o.iterate(1)
        print(kind, n, colours, s.debug_sweeps(), flush=True)
        assert s.debug_sweeps()["redone"] == 0
        assert rel(s.debug_stage("dW"), o.stage("dW")) < TOL
        assert rel(s.debug_stage("Wt"), o.stage("Wt")) < TOL
        assert rel(s.dG.cpu().numpy(), o.stage("dG")) < TOL
    assert s.debug_sweeps()["form"] == form


@pytest.mark.parametrize("kind,n,colours,form", [("hex", 6, 5, "blocks"), ("tet", 6, 13, "blocks"),
                                                 ("hex", 6, 17, "colours"), ("mixed", 5, 18, "colours")])
def test_adjoint_sweeps_of_many_colours(kind, n, colours, form):
    """Transposed macro sweeps: the split colouring against the mesh's own, the same relaxations."""
    import torch
    from paper_2303_10846_amd.binding import Solver
    c = configs.open_box_case(n=n, nv_side=3, kind=kind)
    s = Solver(c, precision="fp64")
    s.init_equilibrium(c["W0"])
    s.iterate(3)
    state = s.get_state()
    m = dict(c, mesh=split_colours(c["mesh"], colours))
    b = Solver(m, precision="fp64")
    b.set_state(*state)
    t = torch.randn(s.nc, 6, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    x, y = (k.debug_adjoint_sweeps(t, True, 5).cpu().numpy() for k in (s, b))
    assert b.debug_sweeps()["form"] == form
    assert rel(y, x) < TOL

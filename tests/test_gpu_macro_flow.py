"""The macroscopic sweeps against the oracle at the edges of their launch forms: one workgroup (up to 16
wavefronts), blocks over up to 256 workgroups, and a launch per colour beyond the largest mesh of 54 000 cells.  A
wavefront holds 16 tetrahedra or 8 cells of 6 face slots of one colour."""
import sys

import numpy as np
import pytest

import oracle
from paper_2303_10846_amd.cases import configs

pytestmark = pytest.mark.gpu

TOL = 1e-11  # the FP64 parity bar of the suite


def colrel(a, b):
    """The suite's metric: max|a - b| per column over that column's largest value, or over the whole array's where
    the column is zero by an identity (below 1e-6 of the array's largest value)."""
    top = float(np.max(np.abs(b)))
    out = 0.0
    for m in range(b.shape[1]):
        col = float(np.max(np.abs(b[:, m])))
        out = max(out, float(np.max(np.abs(a[:, m] - b[:, m]))) / max(col if col >= 1e-6 * top else top, 1e-300))
    return out


@pytest.mark.parametrize("kind,n,nv_side,n_macro", [
    ("hex", 1, 4, 40),     # one cell, one colour, no neighbour
    ("hex", 2, 4, 1),      # two colours, one wavefront each
    ("tet", 3, 4, 0),      # no sweep: dW = 0
    ("hex", 5, 4, 40),     # 16 wavefronts: the largest one-workgroup mesh
    ("hex", 6, 4, 40),     # 28 wavefronts, 216 blocks of one cell
    ("tet", 4, 4, 3),      # three colours, an odd number of pairs
    ("mixed", 5, 4, 40),   # 5- and 6-face cells with unused slots
    ("tet", 11, 3, 40),    # 501 wavefronts
    ("tet", 13, 3, 40),    # 826 wavefronts, 51 cells a block
    ("tet", 14, 3, 40),    # 16 464 cells: blocks of 16 wavefronts
    ("tet", 20, 3, 3),     # 48 000 cells: near the largest mesh in blocks
    ("tet", 21, 3, 3),     # 55 566 cells: a launch per colour
    ("hex", 29, 3, 3),     # 24 389 cells of 6 slots
    ("hex", 7, 4, 2),      # 343 cells: blocks of one and two cells; windows of two periods, the last cut to one step
    ("hex", 8, 4, 3),      # .. and to three steps
    ("hex", 20, 3, 40),    # 8 000 cells, 31 a block
    ("mixed", 8, 3, 40),   # blocks with cells of 5 and 6 faces
    ("tet", 8, 3, 1),      # one pair
])
def test_macro_sweeps_match_oracle(kind, n, nv_side, n_macro):
    from paper_2303_10846_amd.binding import Solver
    c = configs.open_box_case(n=n, nv_side=nv_side, kind=kind)
    num = dict(c["num"], n_macro=n_macro)
    print("case", c["name"], len(c["mesh"].get("cells", c["mesh"].get("tets"))), "cells, pairs", n_macro, flush=True)
    sys.stdout.flush()
    o = oracle.Oracle(c, num=num)
    o.init_equilibrium(c["W0"])
    o.iterate(2)
    G, R, W, q = o.get_state()
    s = Solver(c, precision="fp64", num=num)
    for _ in range(2):  # the second call's versions follow the first's in the same buffer
        s.set_state(G, R, W, q)
        s.iterate(1)
    o.iterate(1)
    assert colrel(s.debug_stage("Fmac"), o.stage("Fmac")) < TOL
    if n_macro:
        assert colrel(s.debug_stage("dW"), o.stage("dW")) < TOL
    else:
        assert not np.any(s.debug_stage("dW"))
    assert colrel(s.debug_stage("Wt"), o.stage("Wt")) < TOL


@pytest.mark.parametrize("kind,n", [("hex", 6), ("tet", 5), ("mixed", 5)])
def test_adjoint_macro_sweeps_in_blocks(kind, n):
    """The transposed sweeps, as a part of the adjoint's preconditioner: the same gradient in fewer iterations."""
    from paper_2303_10846_amd.binding import Solver
    c = configs.open_box_case(n=n, nv_side=5, kind=kind)
    print("case", c["name"], flush=True)
    s = Solver(c, precision="fp64")
    s.init_equilibrium(c["W0"])
    s.iterate(140)
    a = s.adjoint(1, 2, restart=60, max_iter=600, rtol=1e-10)
    ab = s.adjoint(1, 2, restart=60, max_iter=600, rtol=1e-10, macro_pairs=10)
    print("iterations", a["iterations"], ab["iterations"], flush=True)
    assert a["converged"] and ab["converged"] and ab["iterations"] < a["iterations"]
    assert np.allclose(ab["dJdp"], a["dJdp"], rtol=1e-6, atol=0.0)

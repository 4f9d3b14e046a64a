"""Which meshes take the micro sweeps in one launch, on both sides of the rule's lines (workgroups that run at once,
relaxations that pay for the start, a colour's cells), with the increments against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2303_10846_amd.cases import configs

pytestmark = pytest.mark.gpu

# FP64: the parity bar of the suite.  Mixed: the suite's bar of FP32 increments.
TOL = {"fp64": 1e-11, "mixed": 1e-4}


def nrel(a, b):
    return float(np.max(np.abs(np.asarray(a, np.float64) - b)) / max(float(np.max(np.abs(b))), 1e-300))


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind,n,nv_side,n_micro,one", [
    ("hex", 1, 6, 2, False),   # one colour: one relaxation either way
    ("hex", 1, 25, 2, False),  # 15 625 velocities: 3 907 workgroups in turn took 22 us, the launch 6.5
    ("hex", 2, 12, 2, True), ("hex", 2, 13, 2, False),  # 1 728 and 2 197 velocities
    ("tet", 2, 12, 2, True), ("tet", 2, 22, 2, False),
    ("tet", 3, 12, 1, True),
    # beside macro sweeps in blocks:
    ("hex", 7, 8, 1, True), ("hex", 7, 10, 2, True),
    ("hex", 8, 3, 1, False), ("hex", 8, 3, 2, True), ("hex", 8, 11, 10, False),  # 256 cells a colour
    ("tet", 5, 5, 1, True), ("tet", 5, 11, 1, False),  # up to 341: two rounds
    ("hex", 9, 3, 2, False), ("hex", 9, 3, 12, True),
    ("hex", 10, 6, 2, False),
])
def test_micro_sweeps_on_both_sides_of_the_rule(kind, n, nv_side, n_micro, one, precision):
    from paper_2303_10846_amd.binding import Solver
    c = configs.open_box_case(n=n, nv_side=nv_side, kind=kind)
    num = dict(c["num"], n_micro=n_micro, n_macro=2)
    print("case", c["name"], precision, "pairs", n_micro, flush=True)
    o = oracle.Oracle(c, num=num)
    o.init_equilibrium(c["W0"])
    o.iterate(2)
    s = Solver(c, precision=precision, num=num)
    s.set_state(*o.get_state())
    s.profile(True)
    s.iterate(1)
    o.iterate(1)
    colours = int(np.count_nonzero(np.diff(c["mesh"]["color_offsets"])))
    steps = 1 if colours == 1 else 2 * (colours - 1) * n_micro + 1
    assert s.profile_read()["micro"][1] == (1 if one else steps)
    assert nrel(s.dG.cpu().numpy(), o.stage("dG")) < TOL[precision]
    assert nrel(s.dR.cpu().numpy(), o.stage("dR")) < TOL[precision]

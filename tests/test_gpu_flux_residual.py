"""The explicit micro flux with several velocities a lane and with one (an output that is not aligned): against the
oracle in FP64, against each other with FP32 distributions."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_2303_10846_amd.cases import configs

pytestmark = pytest.mark.gpu


def nrel(a, b):
    return float(np.max(np.abs(a - b)) / max(float(np.max(np.abs(b))), 1e-300))


def _grid(nx, ny, nz, half=4.0):
    ax = [(np.arange(n) + 0.5) * (2 * half / n) - half for n in (nx, ny, nz)]
    u = np.stack(np.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)
    return u, np.full(len(u), (2 * half) ** 3 / (nx * ny * nz))


# 1e-11: the FP64 parity bar of the suite; 4e-6: its bar on F with FP32 distributions (sums of terms up to ~10 times
# the result, some tens of units of FP32 rounding)
@pytest.mark.parametrize("kind", ["tet", "hex"])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-11), ("mixed", 4e-6)])
@pytest.mark.parametrize("dims", [(8, 8, 8), (9, 9, 6), (7, 7, 7)])  # nv mod 4: 0, 2, 3
def test_flux_widths(dims, precision, tol, kind):
    from paper_2303_10846_amd.binding import Solver
    u, w = _grid(*dims)
    c = dict(configs.open_box_case(n=3, nv_side=4, kind=kind), u=u, w=w)
    print("case", c["name"], precision, "nv", len(u), flush=True)
    o = oracle.Oracle(c)
    o.init_equilibrium(c["W0"])
    o.iterate(2)
    G, R, W, q = o.get_state()
    s = Solver(c, precision=precision)
    s.set_state(G, R, W, q)
    FG, FR, _ = s.residual()
    t = s.torch
    rows = [t.empty(s.G.numel() + 1, dtype=s.G.dtype, device=s.G.device)[1:].view(s.G.shape) for _ in range(2)]
    Fm = np.empty((s.nc, 6))
    assert s.lib.cis_residual(s.h, *[C.c_void_p(x.data_ptr()) for x in rows],
                              Fm.ctypes.data_as(C.POINTER(C.c_double))) == 0
    o.explicit()
    for a, one, name in ((FG, rows[0], "FG"), (FR, rows[1], "FR")):
        a, one = a.cpu().numpy().astype(np.float64), one.cpu().numpy().astype(np.float64)
        assert nrel(a, one) < tol
        if precision == "fp64":
            assert nrel(a, o.stage(name)) < tol

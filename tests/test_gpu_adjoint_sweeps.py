"""The sweeps of the adjoint's preconditioner by themselves, against a host FP64 implementation of the same coloured
relaxations: a wrong neighbour or a stale value would be hidden behind GMRES, which converges with any
preconditioner.  The transposed macroscopic system in every form (one workgroup, blocks of 8 and of 16 wavefronts, a
launch per colour) and the transposed transport sweeps in one launch and in one per colour."""
import numpy as np
import pytest

import oracle
from paper_2303_10846_amd.cases import configs

pytestmark = pytest.mark.gpu

TOL = 1e-11  # the FP64 parity bar of the suite


def sequence(m, pairs):
    out = []
    for _ in range(pairs):
        for c in list(range(m)) + list(range(m - 1, -1, -1)):
            if not out or out[-1] != c:
                out.append(c)
    return out


def random_W(nc, rng):
    rho = 1.0 + 0.2 * rng.uniform(-1, 1, nc)
    U = 0.4 * rng.uniform(-1, 1, (nc, 3))
    T, Trot = (1.0 + 0.2 * rng.uniform(-1, 1, nc) for _ in range(2))
    eint = 2.5 * rho * 0.5 * T
    return np.column_stack([rho, rho[:, None] * U, eint + 0.5 * rho * (U * U).sum(1), rho * 0.5 * Trot])


class Host:
    """Geometry per cell slot from the oracle: neighbour (-1: none), A/V, A, outward normal, dl."""

    def __init__(self, case):
        self.o = oracle.Oracle(case)
        g = self.o.geometry()
        cf = g["cf"]
        nc = len(cf)
        used = cf >= 0
        f = np.where(used, cf, 0)
        own = g["fo"][f] == np.arange(nc)[:, None]
        nb = np.where(own, g["fn"][f], g["fo"][f])
        self.nb = np.where(used, nb, -1)
        self.V = g["V"]
        self.A = np.where(used, g["A"][f], 0.0)
        self.n = np.where(own[..., None], 1.0, -1.0) * g["n"][f]
        inner = self.nb >= 0
        d = np.where(inner[..., None], g["xc"][np.where(inner, self.nb, 0)], g["xf"][f]) - g["xc"][:, None]
        self.dl = np.sqrt((d * d).sum(-1)) * np.where(inner, 1.0, 2.0)
        off = np.asarray(case["mesh"]["color_offsets"])
        self.cells = [np.arange(off[c], off[c + 1]) for c in range(len(off) - 1) if off[c + 1] > off[c]]
        self.gas = case["gas"]

    def prims(self, W):
        g = self.gas
        rho, U = W[:, 0], W[:, 1:4] / W[:, :1]
        eint = W[:, 4] - 0.5 * rho * (U * U).sum(1)
        T, Ttr = 0.4 * eint / (rho * g["R"]), (2.0 / 3.0) * (eint - W[:, 5]) / (rho * g["R"])
        return rho, U, T, Ttr

    def mu(self, Ttr):
        return self.gas["mu_ref"] * (Ttr / self.gas["T_ref"]) ** self.gas["omega_vhs"]

    def macro(self, W, t, pairs):
        """Mac^T u = t by point relaxations over the colours, from zero."""
        g = self.gas
        rho, U, T, Ttr = self.prims(W)
        j = np.where(self.nb >= 0, self.nb, np.arange(len(W))[:, None])
        mean = lambda x: 0.5 * (x[:, None] + x[j])  # noqa: E731
        r = (np.abs((mean(U) * self.n).sum(-1)) + np.sqrt(g["gamma"] * g["R"] * mean(T)) +
             2.0 * self.mu(mean(Ttr)) / (mean(rho) * np.where(self.A > 0, self.dl, 1.0)))
        D = (0.5 * self.A / self.V[:, None] * r).sum(1)
        tau = self.mu(Ttr) / (rho * g["R"] * Ttr)
        D = np.column_stack([D] * 5 + [D + 1.0 / (g["Z"] * tau)])
        u = np.zeros_like(t)
        for c in sequence(len(self.cells), pairs):
            i = self.cells[c]
            acc = t[i].copy()
            for a in range(self.nb.shape[1]):
                ok = self.nb[i, a] >= 0
                k, uj = i[ok], u[self.nb[i[ok], a]]
                gj = euler_vjp(W[k], self.n[k, a], uj)
                acc[ok] += (0.5 * self.A[k, a] / self.V[self.nb[k, a]])[:, None] * (gj + r[k, a][:, None] * uj)
            u[i] = acc / D[i]
        return u

    def transport(self, W, uvel, x_in, pairs, snap):
        """(D + N^T) x = -in over the colours, from zero; x_in [nc][nv]."""
        rho, _, _, Ttr = self.prims(W)
        tau = self.mu(Ttr) / (rho * self.gas["R"] * Ttr)
        un = np.einsum("iad,kd->iak", self.n, uvel)
        un = np.where(np.abs(un) <= snap * np.sqrt((uvel * uvel).sum(1)), 0.0, un)
        up = np.maximum(un, 0.0) * self.A[..., None]
        D = 1.0 / tau[:, None] + up.sum(1) / self.V[:, None]
        x = np.zeros_like(x_in)
        for c in sequence(len(self.cells), pairs):
            i = self.cells[c]
            acc = -x_in[i]
            for a in range(self.nb.shape[1]):
                nb = self.nb[i, a]
                acc += np.where((nb >= 0)[:, None], up[i, a] / self.V[nb][:, None] * x[nb], 0.0)
            x[i] = acc / D[i]
        return x


def euler_vjp(W, n, v):
    """J^T v of the Euler flux along n with the rotational-energy row, by the complex step."""
    out = np.empty_like(v)
    for m in range(6):
        Wc = W.astype(complex)
        Wc[:, m] += 1e-30j
        U = Wc[:, 1:4] / Wc[:, :1]
        Un = (U * n).sum(1)
        p = 0.4 * (Wc[:, 4] - 0.5 * Wc[:, 0] * (U * U).sum(1))
        G = np.column_stack([Wc[:, 0] * Un, Wc[:, 1:4] * Un[:, None] + p[:, None] * n, (Wc[:, 4] + p) * Un,
                             Wc[:, 5] * Un])
        out[:, m] = (G.imag / 1e-30 * v).sum(1)
    return out


def _setup(kind, n, nv_side):
    from paper_2303_10846_amd.binding import Solver
    c = configs.open_box_case(n=n, nv_side=nv_side, kind=kind)
    rng = np.random.default_rng(7 * n + nv_side)
    s = Solver(c, precision="fp64")
    W = random_W(s.nc, rng)
    s.set_state(np.zeros((s.nc, s.nv)), np.zeros((s.nc, s.nv)), W, np.zeros((s.nc, 6)))
    return c, s, W, rng


@pytest.mark.parametrize("kind,n,pairs,form", [
    ("hex", 1, 2, "workgroup"), ("tet", 3, 3, "workgroup"), ("hex", 5, 10, "workgroup"),
    ("hex", 6, 10, "blocks"), ("tet", 4, 1, "blocks"), ("tet", 6, 10, "blocks"), ("mixed", 5, 3, "blocks"),
    ("hex", 10, 2, "blocks"), ("tet", 14, 3, "blocks"), ("tet", 20, 4, "wide blocks"), ("hex", 29, 3, "wide blocks"),
    ("tet", 21, 3, "colours"),
])
def test_transposed_macro_sweeps(kind, n, pairs, form):
    import torch
    c, s, W, rng = _setup(kind, n, 2)
    t = rng.standard_normal((s.nc, 6))
    print(kind, n, s.nc, "cells, pairs", pairs, flush=True)
    want = Host(c).macro(W, t, pairs)
    x = torch.as_tensor(t).cuda()
    for _ in range(2):  # the second call's tags follow the first's in the same buffer
        got = s.debug_adjoint_sweeps(x, True, pairs).cpu().numpy()
        assert np.max(np.abs(got - want) / np.max(np.abs(want), axis=0)) < TOL
    assert s.debug_sweeps()["form"] == form


@pytest.mark.parametrize("kind,n,nv_side,pairs", [
    ("hex", 1, 4, 2),      # one cell
    ("hex", 2, 3, 1),      # 27 velocities: the last workgroup has 3
    ("tet", 3, 5, 2), ("mixed", 4, 6, 2), ("tet", 5, 5, 3), ("hex", 7, 9, 2),
    ("hex", 8, 5, 2),      # 256 cells a colour
    ("hex", 9, 6, 6),      # more than one round of 256 cells a colour
    ("tet", 6, 4, 2),      # 1 296 cells
    ("tet", 2, 13, 2),     # 2 197 velocities: more workgroups than run at once
])
def test_transposed_transport_sweeps(kind, n, nv_side, pairs):
    import torch
    c, s, W, rng = _setup(kind, n, nv_side)
    P = s.nc * s.nv
    x = rng.standard_normal(2 * P + 12 * s.nc)
    print(kind, n, s.nc, "cells", s.nv, "velocities, pairs", pairs, flush=True)
    got = s.debug_adjoint_sweeps(torch.as_tensor(x).cuda(), False, pairs).cpu().numpy()
    h = Host(c)
    for k in range(2):
        want = h.transport(W, np.asarray(c["u"]), x[k * P:(k + 1) * P].reshape(s.nc, s.nv), pairs, c["num"]["snap"])
        assert np.max(np.abs(got[k * P:(k + 1) * P].reshape(s.nc, s.nv) - want)) < TOL * np.max(np.abs(want))
    assert np.array_equal(got[2 * P:], x[2 * P:])

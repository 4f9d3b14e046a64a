"""The macro sweeps in blocks when a wait of theirs runs out (a workgroup kept off the device): the call goes on with a
launch per colour and its results stay those of an undisturbed call; and the sweeps beside other work on the device."""
import threading

import numpy as np
import pytest

from paper_2303_10846_amd.cases import configs

pytestmark = pytest.mark.gpu

# FP64: the parity bar of the suite.  Mixed: the suite's bar for W after an iteration (FP32 rounding of phi).
TOL = {"fp64": 1e-11, "mixed": 2e-6}


def rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    return float(np.max(np.abs(a - b)) / max(float(np.max(np.abs(b))), 1e-300))


def _solver(kind, n, precision="fp64", nv_side=4, **kw):
    from paper_2303_10846_amd.binding import Solver
    c = configs.open_box_case(n=n, nv_side=nv_side, kind=kind)
    s = Solver(c, precision=precision, **kw)
    s.init_equilibrium(c["W0"])
    return s


@pytest.mark.parametrize("kind,n,form", [
    ("tet", 2, "workgroup"), ("hex", 5, "workgroup"), ("hex", 6, "blocks"), ("tet", 6, "blocks"),
    ("tet", 14, "blocks"), ("tet", 20, "wide blocks"), ("tet", 21, "colours"),
    ("hex", 33, "colours"),  # 35 937 cells of 6 slots: over 128 a block, 16 wavefronts of 8
])
def test_form_of_the_sweeps(kind, n, form):
    s = _solver(kind, n, nv_side=3)
    print(kind, n, s.debug_sweeps(), flush=True)
    s.profile(True)
    s.iterate(2)
    assert s.debug_sweeps()["form"] == form
    launches = s.profile_read()["macro"][1]
    assert launches == 2 if form != "colours" else launches > 2


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind,n,first", [("tet", 4, 0), ("tet", 4, 3), ("hex", 6, 4), ("mixed", 5, 1),
                                          ("tet", 20, 2), ("tet", 3, 0)])
def test_iterations_after_a_wait_ran_out(kind, n, first, precision, noalloc):
    a, b = _solver(kind, n, precision), _solver(kind, n, precision)
    print(kind, n, precision, "waits run out from launch", first, flush=True)
    b.debug_sweeps(polls=0, first=first)
    run = (lambda s, k: s.iterate_noalloc(k)) if noalloc else (lambda s, k: s.iterate(k))
    ha, hb = run(a, 5), run(b, 5)
    waits = a.debug_sweeps()["form"] != "workgroup"
    assert b.debug_sweeps()["redone"] == (1 if waits else 0) and a.debug_sweeps()["redone"] == 0
    assert rel(hb, ha) <= TOL[precision]
    for x, y in zip(b.get_state(), a.get_state()):
        assert rel(x, y) <= TOL[precision]
    b.debug_sweeps(polls=1 << 18)  # and back to one launch, in the same exchange buffer
    assert rel(run(b, 3), run(a, 3)) <= TOL[precision]
    assert b.debug_sweeps()["redone"] == (1 if waits else 0)


@pytest.mark.parametrize("first", [0, 3, 6, 8])  # the first step, one in a cycle, its end, a later cycle
def test_adjoint_after_a_wait_ran_out(first):
    s = _solver("hex", 6, nv_side=5)
    s.iterate(140)
    kw = dict(restart=6, max_iter=600, rtol=1e-10, macro_pairs=10)
    a = s.adjoint(1, 2, **kw)
    s.debug_sweeps(polls=0, first=first)
    b = s.adjoint(1, 2, **kw)
    print("launch", first, "iterations", a["iterations"], b["iterations"], flush=True)
    assert s.debug_sweeps()["redone"] == 1
    assert a["converged"] and b["converged"]
    # both solve to 1e-10; the preconditioner's rounding alone differs
    assert np.allclose(b["dJdp"], a["dJdp"], rtol=1e-6, atol=0.0)
    assert abs(b["iterations"] - a["iterations"]) <= 2


def test_two_states_on_two_streams():
    import torch
    kinds = [("tet", 6), ("hex", 10)]
    ref = [_solver(*k) for k in kinds]
    want = [s.iterate(40) for s in ref]
    streams = [torch.cuda.Stream() for _ in kinds]
    got, solvers = [None, None], []
    for k, st in zip(kinds, streams):
        with torch.cuda.stream(st):
            solvers.append(_solver(*k, stream=st))
    torch.cuda.synchronize()

    def work(i):
        got[i] = np.concatenate([solvers[i].iterate(10) for _ in range(4)])

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(2):
        assert rel(got[i], want[i]) <= TOL["fp64"]
        for x, y in zip(solvers[i].get_state(), ref[i].get_state()):
            assert rel(x, y) <= TOL["fp64"]


def test_sweeps_beside_products_on_another_stream():
    import torch
    a, b = _solver("tet", 6), _solver("tet", 6)
    want = a.iterate(20)
    x = torch.randn(4096, 4096, device="cuda", dtype=torch.float32)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for _ in range(40):
            y = x @ x
    got = b.iterate(20)
    torch.cuda.synchronize()
    assert torch.isfinite(y).all()
    assert rel(got, want) <= TOL["fp64"]


@pytest.mark.parametrize("kind,n", [("tet", 6), ("hex", 6)])
def test_tags_start_again_before_they_run_out(kind, n):
    """The tags of the windows end at 2^31 - 1; the launch that would pass it clears the exchange buffer."""
    a, b = _solver(kind, n), _solver(kind, n)
    a.iterate(2)
    per_launch = a.debug_sweeps()["tag"] // 2
    b.iterate(2)
    # the third launch from here passes the end; then one that ends on it exactly, and the next
    for left in (2 * per_launch + 1, per_launch, per_launch - 1):
        b.debug_sweeps(tag=2**31 - 1 - left)
        assert rel(b.iterate(5), a.iterate(5)) <= TOL["fp64"]
        assert b.debug_sweeps()["redone"] == 0
        assert b.debug_sweeps()["tag"] == (5 - left // per_launch) * per_launch
    for x, y in zip(b.get_state(), a.get_state()):
        assert rel(x, y) <= TOL["fp64"]


def test_blocks_are_laid_out_by_the_first_call_that_sweeps():
    s = _solver("hex", 6, nv_side=5)
    s.residual()
    s.wall_loads(1)
    s.adjoint(1, 2, restart=2, max_iter=2)  # no macro sweeps in its preconditioner
    assert s.debug_sweeps()["form"] == "not laid out"
    s.adjoint(1, 2, restart=2, max_iter=2, macro_pairs=2)
    assert s.debug_sweeps()["form"] == "blocks"
    s = _solver("hex", 6)
    s.iterate_noalloc(1)
    assert s.debug_sweeps()["form"] == "blocks"


@pytest.mark.parametrize("n_macro,n_micro,one", [(40, 2, True), (2, 2, True), (2, 50, False), (40, 50, True),
                                                 (0, 2, False)])
def test_blocks_only_where_they_pay(n_macro, n_micro, one):
    """Launches of a stream start later after the cooperative one: with few macro and many micro sweeps the launches
    per colour are the faster form."""
    import oracle
    from paper_2303_10846_amd.binding import Solver
    c = configs.open_box_case(n=10, nv_side=4, kind="hex")
    num = dict(c["num"], n_macro=n_macro, n_micro=n_micro)
    o = oracle.Oracle(c, num=num)
    o.init_equilibrium(c["W0"])
    s = Solver(c, num=num)
    s.init_equilibrium(c["W0"])
    s.profile(True)
    s.iterate(2)
    o.iterate(2)
    assert s.profile_read()["macro"][1] == (2 if one else 2 * (3 + (2 * n_macro + 1 if n_macro else 0)))
    assert s.debug_sweeps()["form"] == ("blocks" if one else "not laid out")
    for x, y in zip(s.get_state(), o.get_state()):
        assert rel(x, y) <= TOL["fp64"]


@pytest.mark.parametrize("first", [None, 0, 255, 256, 300])
def test_long_calls_run_in_pieces(first):
    """A call of more iterations than one piece (256), undisturbed and with a wait that runs out in either piece."""
    a, b = _solver("hex", 6, nv_side=3), _solver("hex", 6, nv_side=3)
    want = np.concatenate([a.iterate(100), a.iterate(100), a.iterate(100), a.iterate(40)])
    if first is not None:
        b.debug_sweeps(polls=0, first=first)
    b.profile(True)
    got = b.iterate(340)
    assert b.debug_sweeps()["redone"] == (first is not None)
    one = 340 if first is None else first
    assert b.profile_read()["macro"][1] == one + (340 - one) * (3 + 81)
    assert rel(got, want) <= TOL["fp64"]
    for x, y in zip(b.get_state(), a.get_state()):
        assert rel(x, y) <= TOL["fp64"]

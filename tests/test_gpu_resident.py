"""The resident path (a small LP's iterations in one workgroup) against the
launched kernels on the same LP: an explicit kernel choice equal to the
library's own takes the launched path, and both must give the same bits, in
iterates, solve and pushes.  Sizes at the edges of its rules: one row or
column, rows of one and of many lane groups, tiles longer than a chunk of
entries, more than 4,096 columns (operands from memory), matrices just inside
and outside the LDS, and iteration counts that are not a multiple of a check.
The power iteration and the checks run in the workgroup too."""
import numpy as np
import pytest

from paper_2511_13894_amd import lpgen, pdhg

pytestmark = pytest.mark.gpu


def _lps():
    yield "tiny", lpgen.tiny(3)
    yield "free", lpgen.tiny(5, m=9, n=21, with_free=True)
    yield "one_row", lpgen.planted(1, 7, 2, deg=1)
    yield "one_col", lpgen.from_dense(np.array([[1.0], [2.0], [-1.0]]), [1.0, 3.0, 0.0], [1.0], sense="<<<")
    yield "empty_row", lpgen.from_dense(np.array([[1.0, 2.0, 0.0], [0.0, 0.0, 0.0], [0.0, 1.0, 1.0]]), [2.0, 0.0, 1.0],
                                        [1.0, 1.0, 1.0], sense="=<=")
    yield "c0", lpgen.config0(1)
    yield "ineq", lpgen.planted(150, 400, 9, deg=4, ineq_frac=0.5, upper_frac=0.4)
    yield "powerlaw", lpgen.config1(4, 120, 481)
    yield "long_columns", lpgen.planted(300, 90, 6, deg=60, zero_frac=0.3)  # tiles of more than one chunk
    yield "dense_rows", lpgen.planted(40, 900, 7, deg=9)  # lane groups for the dual half
    yield "transport", lpgen.transportation(30, 77, 2)  # row segments, uniform columns
    yield "streamed", lpgen.planted(700, 2500, 8, deg=5)  # the matrix does not fit the LDS
    yield "many_columns", lpgen.planted(300, 4200, 8, deg=3)  # operands from memory
    yield "launched", lpgen.planted(3000, 9000, 8, deg=6)  # outside the rule


LPS = dict(_lps())


def _own_choice(lp, precision):
    """The library's kernel choice of this LP as explicit lanes, which the resident path declines."""
    s = pdhg.Solver(lp, precision=precision)
    t = s.get_timing()
    return {"lanes_at": t.lanes_at, "lanes_a": t.lanes_a}


def _same(a, b):
    for u, v in zip(a, b):
        np.testing.assert_array_equal(u, v)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", sorted(LPS))
def test_resident_equals_launched(name, precision):
    lp = LPS[name]
    print(f"[resident] {name} {precision}: m={lp.m} n={lp.n} nnz={lp.nnz}", flush=True)
    r = pdhg.Solver(lp, precision=precision)
    k = pdhg.Solver(lp, precision=precision, **_own_choice(lp, precision))
    a, b = r.get_scaling(), k.get_scaling()
    assert (a["eta"], a["sigma_est"], a["power_steps"]) == (b["eta"], b["sigma_est"], b["power_steps"])
    for count in (1, 5, 64, 130):
        a, b = r.iterate(count), k.iterate(count)
        assert (a.status, a.iters, a.restarts) == (b.status, b.iters, b.restarts)
        _same(r.get_iterate(), k.get_iterate())
    r = pdhg.Solver(lp, precision=precision, max_iter=4000, push_max_iter=3000)
    k = pdhg.Solver(lp, precision=precision, max_iter=4000, push_max_iter=3000, **_own_choice(lp, precision))
    a, b = r.solve(), k.solve()
    assert (a.status, a.iters, a.restarts, a.pobj) == (b.status, b.iters, b.restarts, b.pobj)
    _same(r.get_solution(), k.get_solution())
    a, b = r.corner_push(3), k.corner_push(3)
    assert (a.status, a.iters, a.restarts, a.n_fix_lower, a.n_fix_upper) == (b.status, b.iters, b.restarts, b.n_fix_lower,
                                                                            b.n_fix_upper)
    _same(r.get_solution(), k.get_solution())
    a, b = r.dual_push(3), k.dual_push(3)
    assert (a.status, a.iters, a.restarts) == (b.status, b.iters, b.restarts)
    _same(r.get_solution(), k.get_solution())


@pytest.mark.parametrize("kw", [{"halpern": 0}, {"check_every": 7}, {"check_every": 1500}, {"use_graph": 0},
                                {"timing": 1}, {"reflect_gamma": 0.5}])
def test_resident_equals_launched_options(kw):
    lp = LPS["ineq"]
    r = pdhg.Solver(lp, max_iter=3000, **kw)
    k = pdhg.Solver(lp, max_iter=3000, **kw, **_own_choice(lp, "fp64"))
    a, b = r.solve(), k.solve()
    assert (a.status, a.iters, a.restarts) == (b.status, b.iters, b.restarts)
    _same(r.get_solution(), k.get_solution())


def test_resident_solve_after_a_restored_state_and_a_new_start():
    lp = LPS["c0"]
    r, k = pdhg.Solver(lp, precision="fp32"), pdhg.Solver(lp, precision="fp32", **_own_choice(lp, "fp32"))
    r.iterate(100)  # between two checks
    k.set_state(r.get_state())
    a, b = r.solve(), k.solve()
    assert (a.status, a.iters, a.restarts) == (b.status, b.iters, b.restarts)
    _same(r.get_solution(), k.get_solution())
    x, y = np.full(lp.n, 0.1), np.full(lp.m, -0.2)
    for s in (r, k):
        s.set_start(x, y)
    a, b = r.solve(), k.solve()
    assert (a.status, a.iters, a.restarts) == (b.status, b.iters, b.restarts)
    _same(r.get_solution(), k.get_solution())


def test_resident_learned_push_and_history():
    lp = LPS["c0"]
    logits = np.random.default_rng(1).standard_normal(lp.n) * 3
    got = []
    for kw in ({}, _own_choice(lp, "fp64")):
        s = pdhg.Solver(lp, record_history=1, **kw)
        a = s.solve()
        f = s.features(5)
        b = s.corner_push_logits(logits, 0.9, 5)
        got.append((a.iters, a.restarts, b.status, b.iters, b.n_learned_fix, b.n_learned_undo, f, *s.get_solution()))
    for u, v in zip(*got):
        np.testing.assert_array_equal(u, v)

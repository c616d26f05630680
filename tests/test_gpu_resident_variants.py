"""Every variant of the one-workgroup path against the launched kernels, bit for
bit.  The plan that verbosity prints says which variant runs, so an LP that no
longer takes its variant fails here.  Variants 1-3 hold columns of up to 8 entries
(512 columns; 2,048; 2,048 with two rounds of rows, mixed precision only), 4 and 5
of up to 4 and 2 (1,024 columns; 4,096 with two rounds of rows).  LPs on both
sides of a variant's edges, rows in tiles and in lane groups, and phases that end
with non-finite values."""
import re

import numpy as np
import pytest

from paper_2511_13894_amd import lpgen, pdhg

pytestmark = pytest.mark.gpu

TILES, GROUPS = "", " of lane groups"
# name: LP, variant and rounds of rows in float64 and in mixed precision (None: launched), how rows are summed
LPS = {
    "512_columns": (lambda: lpgen.planted(200, 512, 4, deg=5), (1, 1), (1, 1), TILES),
    "two_threads_a_row": (lambda: lpgen.planted(60, 500, 3, deg=4), (1, 1), (1, 1), TILES),
    "513_columns": (lambda: lpgen.planted(200, 513, 4, deg=5), (2, 1), (2, 1), TILES),
    "inequalities": (lambda: lpgen.planted(300, 800, 2, deg=5, ineq_frac=0.4, upper_frac=0.3), (2, 1), (2, 1), TILES),
    "eight_threads_a_row": (lambda: lpgen.planted(40, 900, 7, deg=8), (2, 1), (2, 1), GROUPS),
    "512_rows": (lambda: lpgen.planted(512, 1024, 4, deg=4), (2, 1), (2, 1), TILES),
    "513_rows": (lambda: lpgen.planted(513, 1024, 4, deg=4), None, (3, 2), TILES),
    "1024_rows": (lambda: lpgen.planted(1024, 2000, 4, deg=4), None, (3, 2), TILES),
    "1025_rows": (lambda: lpgen.planted(1025, 2000, 4, deg=4), None, None, TILES),
    "2048_columns": (lambda: lpgen.planted(500, 2048, 4, deg=4), None, (3, 2), TILES),
    "2049_columns": (lambda: lpgen.planted(500, 2049, 4, deg=4), None, None, TILES),
    "one_entry_a_column": (lambda: lpgen.planted(400, 1000, 2, deg=1), (4, 1), (4, 1), TILES),
    "1024_short_columns": (lambda: lpgen.planted(300, 1024, 4, deg=2), (4, 1), (4, 1), TILES),
    "1025_short_columns": (lambda: lpgen.planted(300, 1025, 4, deg=2), (5, 1), (5, 1), TILES),
    "two_rounds_of_tiles": (lambda: lpgen.planted(700, 2000, 2, deg=2), (5, 2), (5, 2), TILES),
    "4096_columns": (lambda: lpgen.transportation(64, 64, 3), (5, 2), (5, 2), GROUPS),
    "4160_columns": (lambda: lpgen.transportation(64, 65, 3), None, None, GROUPS),
    "two_segments": (lambda: lpgen.transportation(40, 100, 3), (5, 2), (5, 2), GROUPS),
}


def _runs(capfd, model):
    """How the iterations of the last printed model of that name run."""
    err = capfd.readouterr().err
    found = re.findall(rf"\[pdhg\] {model}: .*; (launched|in one workgroup.*)", err)
    assert found, err
    return found[-1]


def _expected(name, precision):
    _, fp64, fp32, rows = LPS[name]
    v = fp64 if precision == "fp64" else fp32
    return "launched" if v is None else f"in one workgroup, variant {v[0]}, {v[1]} row rounds{rows}"


def _pair(lp, capfd, expected, **kw):
    """The LP with the library's own choice, and with the same kernels named, which are launched."""
    r = pdhg.Solver(lp, verbosity=1, **kw)
    assert _runs(capfd, "model") == expected
    t = r.get_timing()
    k = pdhg.Solver(lp, verbosity=1, lanes_at=t.lanes_at, lanes_a=t.lanes_a, **kw)
    assert _runs(capfd, "model") == "launched"
    return r, k


def _same(a, b):
    for u, v in zip(a, b):
        np.testing.assert_array_equal(u, v)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", sorted(LPS))
def test_variant_equals_launched(name, precision, capfd):
    lp = LPS[name][0]()
    r, k = _pair(lp, capfd, _expected(name, precision), precision=precision, max_iter=2000, push_max_iter=1500)
    a, b = r.get_scaling(), k.get_scaling()
    assert (a["eta"], a["sigma_est"], a["power_steps"]) == (b["eta"], b["sigma_est"], b["power_steps"])
    for count in (1, 62, 70):  # to a check's first iteration, over one, to between two
        a, b = r.iterate(count), k.iterate(count)
        assert (a.status, a.iters, a.restarts) == (b.status, b.iters, b.restarts)
        _same(r.get_iterate(), k.get_iterate())
    for call in (lambda s: s.solve(), lambda s: s.corner_push(3), lambda s: s.dual_push(3)):
        a, b = call(r), call(k)
        assert (a.status, a.iters, a.restarts) == (b.status, b.iters, b.restarts)
        _same(r.get_solution(), k.get_solution())


def test_a_push_takes_the_variant_of_its_free_columns(capfd):
    lp = lpgen.transportation(64, 65, 3)  # too many columns to begin with
    r, k = _pair(lp, capfd, "launched", max_iter=4000, push_max_iter=2000)
    r.solve(), k.solve()
    a = r.corner_push(3)
    assert _runs(capfd, "push on the free columns").startswith("in one workgroup")
    b = k.corner_push(3)
    assert _runs(capfd, "push on the free columns") == "launched"
    assert (a.status, a.iters, a.restarts) == (b.status, b.iters, b.restarts)
    _same(r.get_solution(), k.get_solution())


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", ["512_columns", "513_columns", "1024_short_columns", "eight_threads_a_row"])
def test_a_phase_that_overflows_ends_alike(name, precision, capfd):
    # a step far past 1 / ||A|| grows the iterates until a check sees no finite candidate
    r, k = _pair(LPS[name][0](), capfd, _expected(name, precision), precision=precision, eta_safety=30.0, max_iter=4000)
    a, b = r.solve(), k.solve()
    assert a.status == b.status == pdhg.PDHG_NUMERICAL
    assert (a.iters, a.restarts) == (b.iters, b.restarts)
    _same(r.get_iterate(), k.get_iterate())

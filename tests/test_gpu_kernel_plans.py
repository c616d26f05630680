"""Which kernels run a model, read from the plan that verbosity prints: tiles the
caller names with lanes_* run as tiles, the library's own choice may run them as
waves, and autotune times both.  Tiles and waves give the same bits, at row
lengths on the edges of the waves' rounds and past them, with empty rows, in
tiles of more than one chunk of entries and a last tile that is not full, in
either half and in a batch."""
import re

import numpy as np
import pytest

from oracle import OracleSolver
from paper_2511_13894_amd import lpgen, pdhg

pytestmark = pytest.mark.gpu


def _plan(capfd, model="model"):
    """(primal, dual) as the last plan of `model` names them, and how the iterations run."""
    err = capfd.readouterr().err
    found = re.findall(rf"\[pdhg\] {model}[^:]*:.*primal half: kernel (.*); dual half: kernel ([^;\n]*)(?:; (.*))?", err)
    assert found, err
    return found[-1]


def _edges(G, transposed):
    """Rows for G lanes each, and rows of one entry to bring the mean length to where the library picks their tiles."""
    T = 256 // G
    lens = [0] + [k * G + d for k in (1, 2, 4, 8, 9, 15) for d in (-1, 0, 1)] + [16 * G]
    rng = np.random.default_rng(G)
    short = [n for n in lens if n <= 8 * G]
    # a tile of short rows, one of all kinds, one of more than a chunk of entries, and a part of one
    lens = np.concatenate([rng.choice(short, T), rng.choice(lens, T), rng.choice([14 * G, 16 * G, 15 * G + 1], T),
                           rng.choice(lens, 5)])
    top = {1: 3, 4: 16, 8: 48}[G]
    more = int((lens.sum() - 0.9 * top * len(lens)) / (0.9 * top - 1))
    lens = np.concatenate([lens, np.ones(more, dtype=int)])
    a = np.zeros((len(lens), 16 * G + 40))
    for r, k in enumerate(lens):
        a[r, rng.permutation(a.shape[1])[:k]] = rng.uniform(0.5, 2.0, k) * rng.choice([-1.0, 1.0], k)
    if transposed:
        a = a.T.copy()
    m, n = a.shape
    return lpgen.from_dense(a, a @ rng.uniform(0.0, 1.0, n), rng.uniform(-1.0, 1.0, n), np.zeros(n), np.full(n, 2.0),
                            "=" * m)


def _same(a, b):
    for u, v in zip(a, b):
        np.testing.assert_array_equal(u, v)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("half", ["dual", "primal"])
@pytest.mark.parametrize("G", [1, 4, 8])
def test_waves_of_the_librarys_choice_equal_named_tiles(G, half, precision, capfd):
    lp = _edges(G, half == "primal")
    code = -(256 // G)
    with capfd.disabled():
        print(f"[plans] {code} {half} {precision} m={lp.m} n={lp.n} nnz={lp.nnz}", flush=True)
    w = pdhg.Solver(lp, precision=precision, verbosity=1)
    plan = _plan(capfd)
    assert plan[half == "dual"] == f"{code} as waves" and plan[2] == "launched", plan
    t = w.get_timing()
    k = pdhg.Solver(lp, precision=precision, verbosity=1, lanes_at=t.lanes_at, lanes_a=t.lanes_a)
    plan = _plan(capfd)
    assert plan[half == "dual"] == f"{code}" and "waves" not in plan[half != "dual"], plan
    a, b = w.get_scaling(), k.get_scaling()
    assert (a["sigma_est"], a["power_steps"]) == (b["sigma_est"], b["power_steps"])
    o = OracleSolver(lp)
    # fp64: the bound of the other iterate tests; fp32 rounds the matrix and the differences it sums to 24 bits
    tol = 1e-10 if precision == "fp64" else 1e-4
    for count in (1, 4, 123):
        w.iterate(count)
        k.iterate(count)
        _same(w.get_iterate(), k.get_iterate())
        if count < 10:
            o.iterate(count)
            for u, v in zip(w.get_iterate(), o.iterate_state()):
                assert np.abs(u - v).max() <= tol * max(1.0, np.abs(v).max())
    x, y = w.kkt(), k.kkt()
    assert (x.rp2, x.rd2, x.pobj, x.dobj) == (y.rp2, y.rd2, y.pobj, y.dobj)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_waves_in_both_halves_equal_named_tiles_over_solve_and_pushes(precision, capfd):
    lp = lpgen.planted(1500, 4000, 9, deg=5, ineq_frac=0.3, zero_frac=0.4)
    kw = dict(precision=precision, max_iter=2000, push_max_iter=1500, verbosity=1)
    w = pdhg.Solver(lp, **kw)
    assert _plan(capfd) == ("-64 as waves", "-64 as waves", "launched")
    k = pdhg.Solver(lp, lanes_at=-64, lanes_a=-64, **kw)
    assert _plan(capfd) == ("-64", "-64", "launched")
    for call in (lambda s: s.solve(), lambda s: s.corner_push(3), lambda s: s.dual_push(4)):
        a, b = call(w), call(k)
        assert (a.status, a.iters, a.restarts) == (b.status, b.iters, b.restarts)
        _same(w.get_solution(), k.get_solution())


def test_named_tiles_of_one_half_leave_the_other_to_the_library(capfd):
    lp = lpgen.planted(1500, 4000, 9, deg=5)
    pdhg.Solver(lp, lanes_a=-32, verbosity=1)
    assert _plan(capfd) == ("-64 as waves", "-32", "launched")
    pdhg.Solver(lp, lanes_at=-128, verbosity=1)
    assert _plan(capfd) == ("-128", "-64 as waves", "launched")


@pytest.mark.parametrize("edges", [None, "dual", "primal"])
def test_waves_in_a_batch_equal_named_tiles(edges, capfd):
    lps = [lpgen.planted(150 + 37 * k, 401 + 90 * k, 9 + k, deg=4, ineq_frac=0.5, zero_frac=0.4) for k in range(5)]
    if edges:  # an LP of the rows above: its other half's rows are too long for waves
        lps.append(_edges(4, edges == "primal"))
    kw = dict(max_iter=512, push_max_iter=512, verbosity=1)
    w = pdhg.Batch(lps, **kw)
    at, da, _ = _plan(capfd, "batch")
    assert at.endswith(" as waves") == (edges != "dual") and da.endswith(" as waves") == (edges != "primal"), (at, da)
    k = pdhg.Batch(lps, lanes_at=int(at.split()[0]), lanes_a=int(da.split()[0]), **kw)
    assert _plan(capfd, "batch")[:2] == (at.split()[0], da.split()[0])
    for call in (lambda s: s.solve(), lambda s: s.corner_push(range(len(lps)))):
        for a, b in zip(call(w), call(k)):
            assert (a.status, a.iters, a.restarts) == (b.status, b.iters, b.restarts)
        for i in range(len(lps)):
            _same(w.get_solution(i), k.get_solution(i))


def test_autotune_times_tiles_and_waves(capfd):
    lp = lpgen.planted(1500, 4000, 9, deg=5)
    pdhg.Solver(lp, autotune=1, verbosity=1)
    err = capfd.readouterr().err
    for half in ("primal", "dual"):
        for code in (-32, -64, -128, -256):
            for how in ("", " as waves"):
                # -128 is never the library's choice; rows of more than 16 entries are too long for one lane
                possible = not how or (code != -128 and not (half == "dual" and code == -256))
                assert (f"autotune {half} half: kernel {code}{how} " in err) == possible, (half, code, how, err)
    pdhg.Batch([lp, lpgen.planted(900, 2000, 3, deg=4)], autotune=1, verbosity=1)
    err = capfd.readouterr().err
    for half in ("primal", "dual"):
        for how in ("", " as waves"):
            assert f"autotune batch {half} half: kernel -64{how} " in err, (half, how, err)

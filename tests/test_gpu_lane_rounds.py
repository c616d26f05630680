"""The lane-group products at the edges of their rounds of four and eight entries a
lane: rows of no entry, of less than one round, of exactly one, two and three
and of one entry more or less, neighbours in a wave ending in different
rounds, in both halves, against the oracle."""
import numpy as np
import pytest

from oracle import OracleSolver
from paper_2511_13894_amd import lpgen, pdhg

pytestmark = pytest.mark.gpu


def _lp(lanes, transposed):
    lens = [0] + [k * lanes + d for k in (1, 2, 3, 4, 5, 7, 8, 9, 12, 16, 24) for d in (-1, 0, 1)]
    a = np.zeros((len(lens), max(lens) + 3))
    rng = np.random.default_rng(lanes)
    for r in rng.permutation(len(lens)):
        a[r, rng.permutation(a.shape[1])[:lens[r]]] = rng.uniform(0.5, 2.0, lens[r]) * rng.choice([-1.0, 1.0], lens[r])
    if transposed:
        a = a.T.copy()
    m, n = a.shape
    return lpgen.from_dense(a, a @ rng.uniform(0.0, 1.0, n), rng.uniform(-1.0, 1.0, n), np.zeros(n), np.full(n, 2.0),
                            "=" * m)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("lanes", [1, 2, 4, 8, 16, 32, 64, -4000])
def test_lane_rounds_follow_the_oracle(lanes, precision):
    # fp64: the bound of the other iterate tests.  fp32 rounds the matrix and
    # the differences it sums to 24 bits, at most 2^-24 a term: over 5
    # iterations of rows with up to 1,537 entries of mixed sign, 1e-4.
    tol = 1e-10 if precision == "fp64" else 1e-4
    for transposed in (False, True):
        if lanes == -4000:
            lp, kw = _lp(16, transposed), {"lanes_a": -4000}
        else:
            lp, kw = _lp(lanes, transposed), {"lanes_a": lanes, "lanes_at": lanes}
        print(f"[lane rounds] {lanes} {precision} m={lp.m} n={lp.n}", flush=True)
        g, o = pdhg.Solver(lp, precision=precision, **kw), OracleSolver(lp)
        for t in range(5):
            g.iterate(1)
            o.iterate(1)
            for u, v in zip(g.get_iterate(), o.iterate_state()):
                assert np.abs(u - v).max() <= tol * max(1.0, np.abs(v).max()), t

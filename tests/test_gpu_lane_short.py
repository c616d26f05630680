"""The lane-group products where the wave's shortest or longest row picks another
loop: one or two lanes a row with every row long (pipelined rounds) and with one
short row among them, and wide groups whose rows have at most one entry a lane,
against the oracle."""
import numpy as np
import pytest

from oracle import OracleSolver
from paper_2511_13894_amd import lpgen, pdhg

pytestmark = pytest.mark.gpu


def _lp(lens, transposed, seed):
    rng = np.random.default_rng(seed)
    a = np.zeros((len(lens), max(lens) + 3))
    for r, k in enumerate(lens):
        a[r, rng.permutation(a.shape[1])[:k]] = rng.uniform(0.5, 2.0, k) * rng.choice([-1.0, 1.0], k)
    if transposed:
        a = a.T.copy()
    m, n = a.shape
    return lpgen.from_dense(a, a @ rng.uniform(0.0, 1.0, n), rng.uniform(-1.0, 1.0, n), np.zeros(n), np.full(n, 2.0),
                            "=" * m)


def _cases(lanes):
    rng = np.random.default_rng(lanes)
    if lanes > 2:  # at most one entry a lane, then one row of a second round
        short = list(rng.choice([0, 1, lanes - 1, lanes], 70))
        return [short, short + [lanes + 1]]
    long = [32 * lanes + d for d in (1, 2, lanes, 4 * lanes, 7 * lanes + 1, 8 * lanes, 15 * lanes, 16 * lanes + 1)]
    rows = list(rng.choice(long, 130))  # more than two waves of rows
    return [rows, rows[:40] + [32 * lanes] + rows[40:], rows + [0]]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("lanes", [1, 2, 16, 32, 64])
def test_lane_loops_follow_the_oracle(lanes, precision):
    # the bounds of test_gpu_lane_rounds.py
    tol = 1e-10 if precision == "fp64" else 1e-4
    for lens in _cases(lanes):
        for transposed in (False, True):
            lp = _lp(lens, transposed, lanes)
            print(f"[lane loops] {lanes} {precision} m={lp.m} n={lp.n}", flush=True)
            kw = {"lanes_at": lanes} if transposed else {"lanes_a": lanes}
            g, o = pdhg.Solver(lp, precision=precision, **kw), OracleSolver(lp)
            for t in range(3):
                g.iterate(1)
                o.iterate(1)
                for u, v in zip(g.get_iterate(), o.iterate_state()):
                    assert np.abs(u - v).max() <= tol * max(1.0, np.abs(v).max()), t

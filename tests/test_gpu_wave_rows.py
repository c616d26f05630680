"""Tiles run as waves (short rows, a launch whose waves are resident at once)
against the oracle.  Row lengths at the edges of the lanes' rounds and past
them, empty rows, rows in tiles of more than one chunk of entries, a last tile
that is not full; in either half, the other one running tiles where its rows are
too long for waves."""
import numpy as np
import pytest

from oracle import OracleSolver
from paper_2511_13894_amd import lpgen, pdhg

pytestmark = pytest.mark.gpu


def _edges(lanes, transposed):
    G = 256 // -lanes
    T = 256 // G
    lens = [0] + [k * G + d for k in (1, 2, 4, 8, 9, 15) for d in (-1, 0, 1)] + [16 * G]
    rng = np.random.default_rng(G)
    short = [n for n in lens if n <= 8 * G]
    # a tile of short rows, one of all kinds, one of more than a chunk of entries, and a part of one
    lens = np.concatenate([rng.choice(short, T), rng.choice(lens, T), rng.choice([14 * G, 16 * G, 15 * G + 1], T),
                           rng.choice(lens, 5)])
    a = np.zeros((len(lens), 16 * G + 40))
    for r, k in enumerate(lens):
        a[r, rng.permutation(a.shape[1])[:k]] = rng.uniform(0.5, 2.0, k) * rng.choice([-1.0, 1.0], k)
    if transposed:
        a = a.T.copy()
    m, n = a.shape
    return lpgen.from_dense(a, a @ rng.uniform(0.0, 1.0, n), rng.uniform(-1.0, 1.0, n), np.zeros(n), np.full(n, 2.0),
                            "=" * m)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("lanes", [-32, -64, -128, -256])
def test_waves_follow_the_oracle(lanes, precision):
    # fp64: the bound of the other iterate tests.  fp32 rounds the matrix and
    # the differences it sums to 24 bits, at most 2^-24 a term: 1e-4 over 5
    # iterations of rows with up to 320 entries of mixed sign.
    tol = 1e-10 if precision == "fp64" else 1e-4
    for transposed in (False, True):
        lp = _edges(lanes, transposed)
        print(f"[waves] {lanes} {precision} m={lp.m} n={lp.n} nnz={lp.nnz}", flush=True)
        g, o = pdhg.Solver(lp, precision=precision, lanes_at=lanes, lanes_a=lanes), OracleSolver(lp)
        for t in range(5):
            g.iterate(1)
            o.iterate(1)
            for u, v in zip(g.get_iterate(), o.iterate_state()):
                assert np.abs(u - v).max() <= tol * max(1.0, np.abs(v).max()), t


@pytest.mark.parametrize("lanes", [-32, -64, -128, -256])
def test_waves_in_a_batch_equal_the_lp_alone(lanes):
    # the bounds of the other comparison of a batch with its LPs alone: their
    # scaling adds the same terms in another order
    lps = [_edges(lanes, False), lpgen.planted(150, 401, 9, deg=4, ineq_frac=0.5), _edges(lanes, True)]
    for pick in ([0, 1], [2, 1], [1]):
        kw = dict(lanes_at=lanes, lanes_a=lanes, max_iter=256, eps_rel=1e-12)
        print(f"[waves] batch {lanes} {pick}", flush=True)
        b = pdhg.Batch([lps[k] for k in pick], **kw)
        res = b.solve()
        for i, k in enumerate(pick):
            g = pdhg.Solver(lps[k], **kw)
            r = g.solve()
            assert (r.iters, r.status) == (res[i].iters, res[i].status)
            for u, v in zip(b.get_solution(i)[:2], g.get_solution()[:2]):
                np.testing.assert_allclose(u, v, rtol=1e-9, atol=1e-12)

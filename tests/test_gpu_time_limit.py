"""A time limit stops a phase after the same iterations whether they run in one
workgroup (a small LP) or in launched halves: the clock is read after every
four cycles."""
import numpy as np
import pytest

from paper_2511_13894_amd import lpgen, pdhg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("check_every", [1, 7, 64, 300, 1500])
def test_time_limit_stops_a_small_lp_after_four_cycles(check_every):
    lp = lpgen.planted(200, 500, 3)
    kw = dict(eps_rel=1e-30, time_limit=1e-9, check_every=check_every)
    r = pdhg.Solver(lp, **kw)
    t = r.get_timing()
    k = pdhg.Solver(lp, lanes_at=t.lanes_at, lanes_a=t.lanes_a, **kw)  # launched halves
    for calls in (1, 2):
        a, b = r.solve(), k.solve()
        assert a.status == b.status == pdhg.PDHG_TIME_LIMIT
        assert a.iters == b.iters == calls * 4 * check_every
        for u, v in zip(r.get_iterate(), k.get_iterate()):
            np.testing.assert_array_equal(u, v)

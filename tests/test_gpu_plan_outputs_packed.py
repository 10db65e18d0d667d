"""Departures on either side of the limit at which their trajectories are
packed once their lengths are known, instead of each taking a whole
trajectory's place behind the planner: plans equal the same requests planned
one by one, bit for bit (-m gpu)."""
import numpy as np
import pytest

from paper_2008_03518_amd import scenario as S

pytestmark = pytest.mark.gpu

POINT_BYTES = 4 * 8 + 4                                  # x, y, z, value; action
LIMIT = 8 << 20


@pytest.mark.parametrize("n, packed", [(64, False), (65, True), (80, True)])
def test_departures_equal_single_requests(n, packed):
    from paper_2008_03518_amd import fastmdp as fm
    sc = S.small(seed=2, n_plans=80, n_requests=1)
    sc.cfg.max_steps = 3600
    assert (n * (sc.cfg.max_steps + 1) * POINT_BYTES > LIMIT) == packed
    o, g = sc.requests.origin[0], sc.requests.goal[0]
    rows = (np.arange(n, dtype=np.int32) * 3) % 120
    with fm.context_for(sc, max_slots=80) as ctx:
        plans, _ = ctx.plan_departures(o, g, rows)
        for i, t in enumerate(rows):
            p = ctx.plan_request(o, g, int(t))
            assert p.status == plans[i].status and p.n_points == plans[i].n_points and plans[i].t0 == t, i
            assert np.array_equal(p.points(), plans[i].points()), i
            assert np.array_equal(p.actions(), plans[i].actions()) and np.array_equal(p.values(), plans[i].values()), i

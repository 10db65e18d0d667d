"""Launches of more requests than CUs at the row lengths where the full sweep
stops taking two per CU: plans equal those of the range query (another
kernel), bit for bit (-m gpu)."""
import copy

import numpy as np
import pytest

from paper_2008_03518_amd import scenario as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads, n", [(24, 2048), (24, 2049), (24, 4096), (24, 4097), (64, 4096), (65, 2048), (65, 2049)])
def test_departures_at_the_limits(heads, n):
    """n plans parked in the box, 300 departures of one request."""
    from paper_2008_03518_amd import fastmdp as fm
    cfg = S.cfg_large_actions()
    cfg.n_head, cfg.max_steps, cfg.plan_capacity = heads, 40, 4100
    cfg.climb, cfg.speed = (-5.0, 0.0, 5.0), (40.0,)
    rng = np.random.default_rng(n + heads)
    rows = 360
    pts = rng.uniform((0, 0, 100), (12000, 12000, 900), (n, 3)).astype(np.float32)
    pts[:20] = np.array([5250.0, 5150.0, 500.0]) + rng.uniform(-250, 250, (20, 3)) * (1.0, 1.0, 0.3)
    pts[np.linalg.norm(pts - [4700.0, 4700.0, 500.0], axis=1) < 250.0] = (11900.0, 11900.0, 800.0)   # the origin is clear
    known = S.Plans(np.zeros(n, np.int32), np.full(n, rows, np.int32), np.repeat(pts[:, None], rows, 1).reshape(-1, 3))
    o, g = np.array([4700.0, 4700.0, 500.0]), np.array([5500.0, 5350.0, 480.0])
    at = np.arange(300, dtype=np.int32)
    out = []
    for rq in (0, 1):
        c = copy.deepcopy(cfg)
        c.range_query = rq
        with fm.Context(c, max_slots=300, planner_threads=1024 if rq else 0) as ctx:
            ctx.load_plans(known)
            out.append(ctx.plan_departures(o, g, at))
    assert out[0][1] == out[1][1]
    print([(p.status, p.n_points) for p in out[0][0][:3]], flush=True)
    assert out[0][0][0].n_points > 5
    for q, (a, b) in enumerate(zip(out[0][0], out[1][0])):
        assert a.status == b.status and a.n_points == b.n_points, q
        assert np.array_equal(a.points(), b.points()) and np.array_equal(a.actions(), b.actions()), q
        assert np.array_equal(a.values(), b.values()), q

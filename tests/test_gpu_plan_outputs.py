"""Plans handed out in one go or packed once their lengths are known: the
departures on either side of the limit (8 MiB of whole trajectories) equal
the same requests planned one by one, bit for bit (-m gpu); and a commit's
check of points spread over several workgroups."""
import numpy as np
import pytest

from paper_2008_03518_amd import scenario as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fm():
    from paper_2008_03518_amd import fastmdp
    return fastmdp


@pytest.mark.parametrize("n", [1, 52, 53, 64])
def test_departures_equal_single_requests(fm, n):
    sc = S.small(seed=2, n_plans=80, n_requests=1)
    sc.cfg.max_steps = 3600                              # 44 bytes a point: 52.9 trajectories in 8 MiB
    o, g = sc.requests.origin[0], sc.requests.goal[0]
    rows = (np.arange(n, dtype=np.int32) * 3) % 120
    with fm.context_for(sc, max_slots=64) as ctx:
        plans, chosen = ctx.plan_departures(o, g, rows)
        for i, t in enumerate(rows):
            p = ctx.plan_request(o, g, int(t))
            assert p.status == plans[i].status and p.n_points == plans[i].n_points and plans[i].t0 == t, i
            assert np.array_equal(p.points(), plans[i].points()), i
            assert np.array_equal(p.actions(), plans[i].actions()) and np.array_equal(p.values(), plans[i].values()), i
    assert -1 <= chosen < n


@pytest.mark.parametrize("at", [0, 255, 256, 599])
def test_commit_conflict_at_any_point(fm, at):
    """A known plan crosses a 600-point trajectory at one of its points."""
    cfg = S.cfg_small()
    k = np.arange(600)
    track = np.stack([200.0 + 10.0 * k, np.full(600, 5000.0), np.full(600, 500.0)], 1)
    other = S.Plans(np.array([at], np.int32), np.array([1], np.int32), track[at:at + 1].astype(np.float32))
    with fm.Context(cfg) as ctx:
        ctx.load_plans(other)
        assert not ctx.commit_points(0, track)
        assert ctx.commit_points(700, track)             # clear of it
        assert not ctx.commit_points(700, track)         # and of itself, once in the table
        assert ctx.n_plans == 2

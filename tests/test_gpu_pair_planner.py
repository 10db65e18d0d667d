"""The full sweep's slices, its choice without scoring every action and its
two-requests-per-CU launches, against the range query (another kernel): plans
equal bit for bit (-m gpu).  Row counts around the slices and a chunk of the
staging; more requests than CUs with rows of two chunks."""
import copy

import numpy as np
import pytest

from paper_2008_03518_amd import scenario as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fm():
    from paper_2008_03518_amd import fastmdp
    return fastmdp


def _same(a, b, q):
    assert a.status == b.status and a.n_points == b.n_points, q
    assert np.array_equal(a.points(), b.points()) and np.array_equal(a.actions(), b.actions()), q
    assert np.array_equal(a.values(), b.values()), q


def _with(cfg, rq):
    c = copy.deepcopy(cfg)
    c.range_query = rq
    return c


@pytest.mark.parametrize("make", ["small", "large"])
@pytest.mark.parametrize("n", [0, 1, 2, 3, 20, 64, 127, 1000])
def test_row_counts(fm, n, make):
    """n plans parked along the tracks of four flights (81 and 360 actions)."""
    cfg = S.cfg_small() if make == "small" else S.cfg_large_actions()
    cfg.plan_capacity = 1024
    rng = np.random.default_rng(n)
    o = rng.uniform((200, 200, 200), (9000, 9000, 800), (4, 3))
    g = rng.uniform((200, 200, 200), (9000, 9000, 800), (4, 3))
    f = rng.uniform(0.05, 0.95, (n, 1))
    k = rng.integers(0, 4, n)
    pts = o[k] + f * (g[k] - o[k]) + rng.uniform(-600, 600, (n, 3)) * (1.0, 1.0, 0.3)
    rows = 700
    plans = S.Plans(np.zeros(n, np.int32), np.full(n, rows, np.int32),
                    np.repeat(pts.astype(np.float32)[:, None], rows, 1).reshape(-1, 3))
    out = []
    for rq in (0, 1):
        with fm.Context(_with(cfg, rq)) as ctx:
            ctx.load_plans(plans)
            out.append([ctx.plan_request(o[q], g[q], 0) for q in range(4)])
    for q in range(4):
        _same(out[0][q], out[1][q], q)


@pytest.mark.parametrize("n", [256, 257, 300])
def test_requests_in_pairs(fm, n):
    sc = S.large_actions(seed=5, n_plans=3400, n_requests=n)
    out = []
    for rq in (0, 1):
        sc.cfg = _with(sc.cfg, rq)
        with fm.context_for(sc, max_slots=512) as ctx:
            plans, committed, _ = ctx.plan_fcfs(sc.requests)
            print(ctx.stats(), flush=True)
        out.append((plans, committed))
    assert np.array_equal(out[0][1], out[1][1])
    for q in range(n):
        _same(out[0][0][q], out[1][0][q], q)

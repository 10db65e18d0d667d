"""Features of many states, grouped by row, equal those of the same states in
small calls (one workgroup a state), bit for bit (-m gpu): sizes around the
limit and a chunk, rows outside the table, states that see part of a row,
and more plans near a group's states than its list holds."""
import numpy as np
import pytest

from paper_2008_03518_amd import scenario as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fm():
    from paper_2008_03518_amd import fastmdp
    return fastmdp


def _both(ctx, pos, goal, rows, seqs):
    n = len(rows)
    whole = ctx.features(pos, goal, rows, seqs).numpy()
    for a in range(0, n, 10000):
        b = min(n, a + 10000)
        part = ctx.features(pos[a:b], goal[a:b], rows[a:b], seqs[a:b]).numpy()
        assert np.array_equal(whole[a:b], part), (n, a)


@pytest.mark.parametrize("n", [16383, 16384, 16447, 131072, 131137])
def test_grouped_equals_single(fm, n):
    sc = S.small(seed=6, n_plans=150, n_requests=12)
    rng = np.random.default_rng(n)
    with fm.context_for(sc) as ctx:
        for q in range(sc.requests.n):                   # entries with sequence numbers
            p = ctx.plan_request(sc.requests.origin[q], sc.requests.goal[q], 0)
            if p.status == fm.OK:
                ctx.commit_plan(p)
        pos = rng.uniform((0, 0, 100), (10000, 10000, 900), (n, 3))
        goal = rng.uniform((0, 0, 100), (10000, 10000, 900), (n, 3))
        goal[::97] = pos[::97]                            # no direction
        rows = rng.integers(-3, 300, n).astype(np.int32)
        rows[::101] = sc.cfg.max_rows + 5
        seqs = rng.integers(0, ctx.next_seq() + 1, n).astype(np.int32)
        _both(ctx, pos, goal, rows, seqs)


def test_crowded_row(fm):
    """200 plans parked around the states of one row."""
    cfg = S.cfg_small()
    rng = np.random.default_rng(1)
    pts = (np.array([5000.0, 5000.0, 500.0]) + rng.uniform(-500, 500, (200, 3))).astype(np.float32)
    plans = S.Plans(np.zeros(200, np.int32), np.full(200, 3, np.int32), np.repeat(pts[:, None], 3, 1).reshape(-1, 3))
    n = 16384
    with fm.Context(cfg) as ctx:
        ctx.load_plans(plans)
        pos = np.array([5000.0, 5000.0, 500.0]) + rng.uniform(-50, 50, (n, 3))
        goal = rng.uniform(100, 900, (n, 3))
        _both(ctx, pos, goal, np.ones(n, np.int32), np.zeros(n, np.int32))

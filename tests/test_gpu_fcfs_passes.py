"""The acceptance passes of the concurrent engine at the edges of their lists
and blocks: the engine's plans equal sequential planning and commits bit for
bit, with requests that withdraw one another's entries (-m gpu).

Request counts around a wave, a workgroup and a launch's worth of prepared
rows; trajectories across several row blocks; a start row at a block's edge;
terrain (refused trajectories withdraw whole); full sweep, range query and
the lookahead window.
"""
import numpy as np
import pytest

from paper_2008_03518_amd import scenario as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fm():
    from paper_2008_03518_amd import fastmdp
    return fastmdp


def _check(fm, sc, t0=0, **kw):
    sc.requests.t0[:] = t0
    with fm.context_for(sc) as ctx:
        seq = []
        for q in range(sc.requests.n):
            p = ctx.plan_request(sc.requests.origin[q], sc.requests.goal[q], t0)
            seq.append((p, ctx.commit_plan(p) if p.status == fm.OK else False))
    with fm.context_for(sc, **kw) as ctx:
        plans, committed, _ = ctx.plan_fcfs(sc.requests)
        st = ctx.stats()
    print(f"{sc.requests.n} requests, {kw}: {st}, committed {int(committed.sum())}", flush=True)
    for q, ((p, c), b, cb) in enumerate(zip(seq, plans, committed)):
        assert p.status == b.status and p.n_points == b.n_points, q
        assert np.array_equal(p.points(), b.points()) and np.array_equal(p.actions(), b.actions()), q
        assert np.array_equal(p.values(), b.values()), q
        assert c == cb, q
    return st


@pytest.mark.parametrize("rq", [0, 1])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 257])
def test_request_counts(fm, n, rq):
    sc = S.small(seed=40 + n, n_plans=60, n_requests=n)
    sc.cfg.range_query = rq
    sc.cfg.plan_capacity = 2048
    st = _check(fm, sc, max_slots=max(n, 2), steps_per_launch=16)
    assert n < 257 or st["resumes"] > 0                  # requests did withdraw entries


@pytest.mark.parametrize("t0", [63, 64, 65])
def test_row_block_edges(fm, t0):
    sc = S.small(seed=3, n_plans=120, n_requests=90)
    sc.cfg.range_query = 1
    sc.cfg.plan_capacity = 2048
    _check(fm, sc, t0=t0, max_slots=33, steps_per_launch=64)


def test_window(fm):
    sc = S.small(seed=9, n_plans=60, n_requests=130)
    sc.cfg.lookahead = 3
    sc.cfg.plan_capacity = 2048
    _check(fm, sc, max_slots=130, steps_per_launch=16)

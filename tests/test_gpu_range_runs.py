"""The range-query planner's runs, detour batches and row grids where they can
go wrong, against the full sweep (which the rest of the suite compares with
the FP64 oracle): plans, actions and values equal bit for bit (-m gpu).

Ties between climbs, between the headings beside a blocked one and at a wide
tie band; a flight along the edge of a well (nearest distances within 1 mm
of the radius, step after step); flights along a wall of the box; wells too
weak to rule out the actions inside; boxes too small for the 16-bit box
test; one heading; terrain; a row's grid after loads, commits, rewinds and a
table read back.
"""
import copy
import os

import numpy as np
import pytest

from paper_2008_03518_amd import scenario as S

pytestmark = pytest.mark.gpu

THREADS = (0, 256, 512)


@pytest.fixture(scope="module")
def fm():
    from paper_2008_03518_amd import fastmdp
    return fastmdp


def _same(a, b, q):
    assert a.status == b.status and a.n_points == b.n_points, q
    assert np.array_equal(a.points(), b.points()) and np.array_equal(a.actions(), b.actions()), q
    assert np.array_equal(a.values(), b.values()), q


def _parked(pts, rows):
    """Plans that stay at the given points for `rows` rows."""
    pts = np.asarray(pts, dtype=np.float32).reshape(-1, 3)
    n = len(pts)
    return S.Plans(np.zeros(n, np.int32), np.full(n, rows, np.int32), np.repeat(pts[:, None, :], rows, 1).reshape(-1, 3))


def _moving(start, step, rows):
    k = np.arange(rows)[:, None]
    return S.Plans(np.zeros(1, np.int32), np.array([rows], np.int32),
                   (np.asarray(start, float)[None] + k * np.asarray(step, float)[None]).astype(np.float32))


def _compare(fm, cfg, plans, flights, terrain=None, tie_rel=None):
    """Each (origin, goal, row) planned by the full sweep and the range query."""
    kw = {} if tie_rel is None else dict(tie_rel=tie_rel)
    out = []
    for rq, th in [(0, 0)] + [(1, t) for t in THREADS]:
        c = copy.deepcopy(cfg)
        c.range_query = rq
        with fm.Context(c, planner_threads=th, **kw) as ctx:
            ctx.load_plans(plans)
            if terrain is not None:
                ctx.set_terrain(terrain)
            out.append([ctx.plan_request(o, g, t) for o, g, t in flights])
    for th, plans_r in zip(THREADS, out[1:]):
        for q, (a, b) in enumerate(zip(out[0], plans_r)):
            _same(a, b, (th, q))
    print([(p.status, p.n_points) for p in out[0]], flush=True)
    return out[0]


def _crossing(rng, n, box, z=(100.0, 900.0)):
    return [(np.array([rng.uniform(0.02, 0.98) * box, rng.uniform(0.02, 0.98) * box, rng.uniform(*z)]),
             np.array([rng.uniform(0.02, 0.98) * box, rng.uniform(0.02, 0.98) * box, rng.uniform(*z)]), int(t))
            for t in rng.integers(0, 40, n)]


def test_ties_between_climbs(fm):
    """The goal lies half a climb step above or below a reachable altitude:
    two climbs are equally near it, step after step."""
    cfg = S.cfg_large_actions()
    plans = _parked([[20000.0, 20000.0, 500.0]], 10)
    o = np.array([2000.0, 3000.0, 400.0])
    p = _compare(fm, cfg, plans, [(o, np.array([6000.0, 3000.0, z]), 0) for z in (400.625, 399.375, 430.625, 400.0)])
    assert all(x.status == fm.OK for x in p)


@pytest.mark.parametrize("off", [0.0, 1e-7, 3.0])
def test_ties_between_headings_beside_a_plan(fm, off):
    """A plan parked on the track: the headings on both sides are equally near
    the goal (exactly, nearly, not)."""
    cfg = S.cfg_large_actions()
    plans = _parked([[5000.0, 3000.0 + off, 400.0], [5600.0, 3000.0, 400.0]], 900)
    o = np.array([2000.0, 3000.0, 400.0])
    _compare(fm, cfg, plans, [(o, np.array([9000.0, 3000.0, 400.0]), 0), (o, np.array([9000.0, 3000.0, 460.0]), 0)])


@pytest.mark.parametrize("gap", [149.9995, 150.0, 150.0004, 150.002, 149.0])
def test_along_the_edge_of_a_well(fm, gap):
    """A plan flies beside the request at its speed, `gap` metres off."""
    cfg = S.cfg_large_actions()
    step = max(cfg.speed) * cfg.dt
    plans = _moving([2000.0, 3000.0 + gap, 400.0], [step, 0.0, 0.0], 400)
    o = np.array([2000.0, 3000.0, 400.0])
    _compare(fm, cfg, plans, [(o + [0.0, -30.0, 0.0], np.array([9000.0, 3000.0, 400.0]), 0),
                              (o + [-400.0, -2.0, 0.0], np.array([9000.0, 3000.0, 400.0]), 3)])


def test_along_the_walls(fm):
    cfg = S.cfg_small()
    rng = np.random.default_rng(3)
    plans = _parked(np.stack([rng.uniform(0, 10000, 120), rng.uniform(0, 400, 120), rng.uniform(100, 900, 120)], 1), 700)
    fl = [(np.array([300.0, y, z]), np.array([9700.0, y, z]), 0) for y in (0.0, 5.0, 160.0) for z in (0.0, 500.0, 1000.0)]
    _compare(fm, cfg, plans, fl)


@pytest.mark.parametrize("change", [dict(r_intr=0.015), dict(r_goal=0.0), dict(n_head=1), dict(n_head=2),
                                    dict(climb=(0.0,), speed=(30.0,)), dict(climb=(-5.0, 5.0), speed=(20.0, 40.0)),
                                    dict(R_intr=40.0), dict(gamma=0.6)])
def test_other_constants(fm, change):
    sc = S.small(seed=31, n_plans=140)
    for k, v in change.items():
        setattr(sc.cfg, k, v)
    _compare(fm, sc.cfg, sc.plans, _crossing(np.random.default_rng(7), 6, 10000.0))


def test_wide_tie_band(fm):
    """A tie band of 1 % holds many actions: every step is decided singly."""
    sc = S.small(seed=32, n_plans=140)
    _compare(fm, sc.cfg, sc.plans, _crossing(np.random.default_rng(8), 3, 10000.0), tie_rel=1e-2)


@pytest.mark.parametrize("box", [500.0, 1500.0])
def test_small_boxes(fm, box):
    cfg = S.cfg_small()
    cfg.box_max = (box, box, 1000.0)
    rng = np.random.default_rng(9)
    pts = np.stack([rng.uniform(0, box, 30), rng.uniform(0, box, 30), rng.uniform(0, 300, 30)], 1)
    _compare(fm, cfg, _parked(pts, 200), _crossing(rng, 8, box, z=(500.0, 900.0)) + _crossing(rng, 8, box, z=(100.0, 900.0)))


def test_terrain(fm):
    sc = S.paper_scale(seed=5, n_plans=700, n_requests=8)
    r = sc.requests
    _compare(fm, sc.cfg, sc.plans, [(r.origin[q], r.goal[q], 0) for q in range(r.n)], terrain=sc.terrain)


def test_grid_follows_the_table(fm, tmp_path):
    """The same loads, commits, rewinds and reads on both planners, with
    requests planned in between: rows with and without a grid, with later
    columns, cut back below and above the indexed ones."""
    sc = S.large_actions(seed=41, n_plans=1500, n_requests=1)
    rng = np.random.default_rng(42)
    more = S.make_known_plans(np.random.default_rng(43), sc.cfg, 500)
    small = S.make_known_plans(np.random.default_rng(44), sc.cfg, 60)
    fl = _crossing(rng, 3, 30000.0)
    tracks = [np.linspace(rng.uniform(0, 30000, 3) * [1, 1, 0.03], rng.uniform(0, 30000, 3) * [1, 1, 0.03], 300)
              for _ in range(12)]
    ref = None
    for rq, th in [(0, 0)] + [(1, t) for t in THREADS]:
        sc.cfg.range_query = rq
        got = []

        def fly(ctx):
            got.append([ctx.plan_request(o, g, t) for o, g, t in fl])

        with fm.Context(sc.cfg, max_slots=8, planner_threads=th) as ctx:
            ctx.load_plans(small)
            fly(ctx)                                   # rows below the grid's threshold
            ctx.snapshot()
            ctx.load_plans(sc.plans)
            fly(ctx)                                   # indexed
            ctx.load_plans_noalloc(more)
            fly(ctx)                                   # many later columns: indexed again
            ctx.snapshot()
            done = [ctx.commit_points(5, t) for t in tracks]
            fly(ctx)                                   # a few later columns
            path = os.path.join(str(tmp_path), f"t{rq}{th}")
            ctx.save_table(path)
            ctx.rewind()
            fly(ctx)                                   # cut back to the indexed columns
            ctx.load_table(path)
            fly(ctx)
            ctx.snapshot()
            reqs = S.make_requests(np.random.default_rng(45), sc.cfg, 6, sc.plans)
            plans, committed, _ = ctx.plan_fcfs(reqs)
            got.append(plans)
            fly(ctx)
            ctx.rewind()
            fly(ctx)
        with fm.Context(sc.cfg, planner_threads=th) as ctx:
            ctx.load_plans(sc.plans)
            fly(ctx)
            ctx.rewind()                               # no snapshot: empties the table
            ctx.load_plans(more)
            fly(ctx)                                   # a grid of dropped entries must not be read
        if ref is None:
            ref = (got, done, committed.tolist())
            print([[(p.status, p.n_points) for p in x] for x in got], done, flush=True)
            continue
        assert (done, committed.tolist()) == ref[1:]
        for k, (x, y) in enumerate(zip(ref[0], got)):
            for q, (a, b) in enumerate(zip(x, y)):
                _same(a, b, (th, k, q))

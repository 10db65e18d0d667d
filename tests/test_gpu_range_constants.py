"""Constants at the ends of what a context takes, through every planner (-m
gpu)."""
import copy

import numpy as np
import pytest

from paper_2008_03518_amd import scenario as S

pytestmark = pytest.mark.gpu


def _plans(cfg, known, flights, terrain=None):
    """Each flight by the full sweep and the range query's planners; and the
    range query's pair counts, with the workgroup size."""
    from paper_2008_03518_amd import fastmdp as fm
    out, pairs = [], []
    for rq, th in ((0, 0), (1, 1024), (1, 256), (1, 512)):
        c = copy.deepcopy(cfg)
        c.range_query = rq
        with fm.Context(c, planner_threads=th) as ctx:
            ctx.load_plans(known)
            if terrain is not None:
                ctx.set_terrain(terrain)
            out.append([])
            for f in flights:
                out[-1].append(ctx.plan_request(*f))
                if rq:
                    pairs.append((th, ctx.stats()["pairs"]))
    return out, pairs


def _same(a, b):
    assert a.status == b.status and a.n_points == b.n_points
    assert np.array_equal(a.points(), b.points()) and np.array_equal(a.actions(), b.actions())
    assert np.array_equal(a.values(), b.values())


def test_flight_into_the_surface():
    """The terrain well ends below the surface: no penalty leads the flight
    around the ridge, and a successor below the surface rejects it."""
    from paper_2008_03518_amd import fastmdp as fm
    cfg = S.cfg_large_actions()
    cfg.R_terr = -20.0
    h = np.zeros((31, 31), np.float32)
    h[:, 5] = 420.0                                      # a ridge across the track, its crest 30 m above the flight
    ter = S.Terrain(31, 31, h, 0.0, 0.0, 1000.0, np.zeros((0, 4)))
    o, g = np.array([2000.0, 3000.0, 390.0]), np.array([9000.0, 3000.0, 390.0])
    known = S.Plans(np.zeros(1, np.int32), np.array([1], np.int32), np.array([[20000.0, 20000.0, 800.0]], np.float32))
    out, _ = _plans(cfg, known, [(o, g, 0)], ter)
    with fm.Context(cfg) as ctx:                         # step by step: the rule scored in full
        ctx.load_plans(known)
        ctx.set_terrain(ter)
        want = ctx.plan_batch(S.Requests(np.zeros(1, np.uint64), o[None], g[None], np.zeros(1, np.int32)))[0]
    assert want.status == fm.REJECT_TERRAIN
    for plans in out:
        _same(want, plans[0])


@pytest.mark.parametrize("at", [0.0, 2.5e7])
def test_entries_at_the_staging_radius(at):
    """Plans that fly ahead and behind at the staging radius less 0 to 2 m,
    in a box whose coordinates FP32 holds to 2 m (the flight's lie almost 1 m
    off theirs): every planner counts the same entries within the radius."""
    cfg = S.cfg_large_actions()
    cfg.R_intr = 151.0
    cfg.box_min, cfg.box_max = (at, at, 0.0), (at + 10000.0, at + 10000.0, 1500.0)
    step = max(cfg.speed) * cfg.dt
    reach = max(cfg.R_intr, cfg.R_sep) + 2.0 + np.hypot(max(cfg.speed), max(cfg.climb)) * cfg.dt
    o, g = np.array([at + 1000.95, at + 3000.0, 400.0]), np.array([at + 9000.0, at + 3000.0, 400.0])
    rows = 380
    k = np.arange(rows)[:, None]
    tracks = [o + [d, 0.0, 0.0] + (k - 1) * np.array([step, 0.0, 0.0])     # at row t + 1, d off the state at row t
              for e in np.linspace(-0.1, 2.0, 12) for d in (reach - e, e - reach)]
    known = S.Plans(np.zeros(len(tracks), np.int32), np.full(len(tracks), rows, np.int32),
                    np.concatenate(tracks).astype(np.float32))
    out, pairs = _plans(cfg, known, [(o, g, 0)])
    for plans in out[1:]:
        _same(out[0][0], plans[0])
    print(pairs, flush=True)
    assert pairs[0][1] > 0 and all(p == pairs[0][1] for _, p in pairs)

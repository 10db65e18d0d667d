"""The range-query planner on a table whose reading from a file broke off: the
rows read so far hold the file's points, and the planner's copies of them (the
grids, the 16-bit coordinates) must hold them as well: plans equal the
1024-thread kernel's, which reads the table itself (-m gpu)."""
import numpy as np
import pytest

from paper_2008_03518_amd import scenario as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_plans", [60, 900])           # rows below the grids' threshold; indexed rows
def test_plans_after_a_table_read_breaks_off(tmp_path, n_plans):
    from paper_2008_03518_amd import fastmdp as fm
    sc = S.large_actions(seed=51, n_plans=n_plans, n_requests=1)
    sc.cfg.range_query = 1
    other = S.make_known_plans(np.random.default_rng(52), sc.cfg, n_plans)
    path = str(tmp_path / "other")
    with fm.Context(sc.cfg) as ctx:
        ctx.load_plans(other)
        ctx.save_table(path)
    with open(path, "r+b") as f:                         # most of the rows, then the file ends
        f.truncate(f.seek(0, 2) * 3 // 4)
    # flights along tracks of the file's plans and of the table's own
    fl = []
    for p in (other, sc.plans):
        off = p.offsets()
        for j in range(3):
            a = p.xyz[off[j]:off[j + 1]].astype(float)
            fl.append((a[min(5, len(a) - 1)] + [0.0, 20.0, 0.0], a[-1], int(p.t0[j]) + 3))
    got = []
    for th in (1024, 0, 256):
        with fm.Context(sc.cfg, planner_threads=th) as ctx:
            ctx.load_plans(sc.plans)
            ctx.plan_request(*fl[0])                     # the table indexed
            with pytest.raises(fm.FastMDPError) as ei:
                ctx.load_table(path)
            assert ei.value.code == fm.E_IO
            got.append([ctx.plan_request(*f) for f in fl])
    print([(p.status, p.n_points) for p in got[0]], flush=True)
    for plans in got[1:]:
        for q, (a, b) in enumerate(zip(got[0], plans)):
            assert a.status == b.status and a.n_points == b.n_points, q
            assert np.array_equal(a.points(), b.points()) and np.array_equal(a.actions(), b.actions()), q
            assert np.array_equal(a.values(), b.values()), q


def test_points_past_the_row_count_follow_too(tmp_path):
    """A file that breaks off replaces points past the counts of a table that
    holds fewer; a rewind to a snapshot with more brings those back."""
    from paper_2008_03518_amd import fastmdp as fm
    sc = S.large_actions(seed=53, n_plans=60, n_requests=1)
    sc.cfg.range_query = 1
    other = S.make_known_plans(np.random.default_rng(54), sc.cfg, 60)
    path, empty = str(tmp_path / "other"), str(tmp_path / "empty")
    with fm.Context(sc.cfg) as ctx:
        ctx.save_table(empty)
        ctx.load_plans(other)
        ctx.save_table(path)
    with open(path, "r+b") as f:
        f.truncate(f.seek(0, 2) * 3 // 4)
    off = other.offsets()
    fl = []
    for j in range(12):                                  # head-on against the file's plans
        a = other.xyz[off[j]:off[j + 1]].astype(float)
        fl.append((a[min(200, len(a) - 1)], a[0], int(other.t0[j])))
    got = []
    for th in (1024, 0, 256):
        with fm.Context(sc.cfg, planner_threads=th) as ctx:
            ctx.load_plans(sc.plans)
            ctx.snapshot()
            ctx.load_table(empty)
            with pytest.raises(fm.FastMDPError):
                ctx.load_table(path)
            ctx.rewind()
            got.append([ctx.plan_request(*f) for f in fl])
    print([(p.status, p.n_points) for p in got[0]], flush=True)
    for plans in got[1:]:
        for q, (a, b) in enumerate(zip(got[0], plans)):
            assert a.status == b.status and a.n_points == b.n_points, q
            assert np.array_equal(a.points(), b.points()) and np.array_equal(a.values(), b.values()), q

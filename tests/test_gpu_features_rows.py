"""Features of many states in few rows, where a wave counts its states of a
row together: bit for bit those of the same states in small calls (-m gpu)."""
import numpy as np
import pytest

from paper_2008_03518_amd import scenario as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shares", [(1,), (63, 1), (8, 7, 49), (1,) * 64, (16,) * 4, (13,) * 5, (9,) * 7 + (1,)])
def test_states_in_few_rows(shares):
    """`shares`: of every 64 states, in one wave, how many lie in each row."""
    from paper_2008_03518_amd import fastmdp as fm
    sc = S.small(seed=8, n_plans=150)
    n = 16447
    rng = np.random.default_rng(len(shares))
    pattern = np.repeat(np.arange(len(shares)), shares)
    rows = np.resize(pattern, n).astype(np.int32) * 3
    for a in range(0, n, 64):                             # in any order within the wave
        rng.shuffle(rows[a:a + 64])
    pos = rng.uniform((0, 0, 100), (10000, 10000, 900), (n, 3))
    goal = rng.uniform((0, 0, 100), (10000, 10000, 900), (n, 3))
    seqs = np.zeros(n, np.int32)
    with fm.context_for(sc) as ctx:
        whole = ctx.features(pos, goal, rows, seqs).numpy()
        for a in range(0, n, 10000):
            b = min(n, a + 10000)
            assert np.array_equal(whole[a:b], ctx.features(pos[a:b], goal[a:b], rows[a:b], seqs[a:b]).numpy()), a

"""The trimming of Odd's own region (csrc/pg_oddregion.hip) where its removal
lists matter: chains longer than one thread follows, vertices that free more
successors than a thread stacks, nothing to trim, everything trimmed."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import odd_region
from paper_1705_02313_amd.pg import Game
from tests.test_gpu_odd_region import _check

pytestmark = pytest.mark.gpu


def _game(rows, owner, pri):
    off = np.zeros(len(rows) + 1, np.int64)
    off[1:] = np.cumsum([len(r) for r in rows])
    return {"n": len(rows), "m": int(off[-1]), "offsets": off,
            "targets": np.concatenate(rows).astype(np.int32),
            "owner": np.asarray(owner, np.uint8),
            "pri": np.asarray(pri, np.int32)}


def _tail(n, top, seed):
    """n Odd vertices in a line into a 3-cycle whose top priority is odd or
    even; an Even vertex watches the line's start."""
    rng = np.random.default_rng(seed)
    rows = [[i + 1] for i in range(n)] + [[n + 1], [n + 2], [n]] + [[0, n]]
    pri = rng.permutation(n + 4) + 10
    pri[n + 1] = 2 * n + 20 + top
    return _game(rows, [1] * (n + 3) + [0], pri)


def _fan(n, seed):
    """A source frees n vertices at once, each of which frees two more, all
    into odd or even loops; some vertices have repeated edges."""
    rng = np.random.default_rng(seed)
    rows = [[1 + i for i in range(n)] * 2]
    for i in range(n):
        rows.append([n + 1 + 2 * i, n + 2 + 2 * i])
    base = 3 * n + 1
    for i in range(2 * n):
        rows.append([base + i % 7] * (1 + i % 2))
    for i in range(7):
        rows.append([base + i])
    rows.append([0])
    return _game(rows, [1] * (len(rows) - 1) + [0],
                 rng.permutation(len(rows)))


CASES = {
    "tail_odd": lambda: _tail(2500, 1, 1),
    "tail_even": lambda: _tail(2500, 0, 2),
    "tail_short": lambda: _tail(1024, 1, 3),
    "fan_in_stack": lambda: _fan(17, 4),
    "fan_past_stack": lambda: _fan(300, 5),
    "cycle_only": lambda: _tail(0, 1, 6),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_trimmed_regions_equal_the_oracle(name):
    g = CASES[name]()
    ref = odd_region.solve(g)
    with Game.from_dict(g, odd_region=True) as d:
        _check(g, d.solve(), ref)

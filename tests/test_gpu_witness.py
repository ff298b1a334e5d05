"""X, the Odd vertices that can stay among Odd vertices (the load's dummies):
sweeps past one group, many members with the same witness, nothing or
everything leaving X, at a size that is no multiple of a word or a block."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import orc
from paper_1705_02313_amd import synth
from paper_1705_02313_amd.pg import Game
from tests.helpers import to_np

pytestmark = pytest.mark.gpu

N = 7001   # past the sizes that load in one block


def _game(rows, owner, seed):
    off = np.zeros(len(rows) + 1, np.int64)
    off[1:] = np.cumsum([len(r) for r in rows])
    return {"n": len(rows), "m": int(off[-1]), "offsets": off,
            "targets": np.concatenate(rows).astype(np.int32),
            "owner": np.asarray(owner, np.uint8),
            "pri": np.random.default_rng(seed).permutation(len(rows))
                     .astype(np.int32)}


def _line(length, seed):
    """An Odd line of `length` into an Even vertex: it leaves X one by one;
    the rest is an Odd cycle whose vertices also lead into the line."""
    rows = [[i + 1] for i in range(length)] + [[0]]
    own = [1] * length + [0]
    k = N - len(rows)
    base = len(rows)
    for i in range(k):
        rows.append(sorted([i % length, base + (i + 1) % k]))
        own.append(1)
    return _game(rows, own, seed)


def _star(members, seed):
    """`members` vertices whose first Odd successor is one that leaves X; two
    in three of them have another."""
    rows, own = [[1], [0]], [1, 0]
    base = 2
    for i in range(N - 2):
        r = [0] if i < members else [base + i]
        if i % 3 and i < members:
            r.append(base + members + i % 5)
        rows.append(r)
        own.append(1)
    return _game(rows, own, seed)


CASES = {
    "line_short": lambda: _line(5, 1),
    "line_mid": lambda: _line(200, 2),
    "line_long": lambda: _line(900, 3),
    "star": lambda: _star(500, 4),
    "star_wide": lambda: _star(3000, 5),
    "none_leaves": lambda: _star(0, 6),
    "all_leave": lambda: _game([[i + 1] for i in range(N)] + [[0]],
                               [1] * N + [0], 7),
    "random": lambda: synth.random_game(N, 2, 3, 8),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_dummies_equal_the_oracle(name):
    g = CASES[name]()
    aug = orc.preprocess(g)
    ref = orc.solve(g)
    with Game.from_dict(g) as d:
        out = d.solve()
        assert out["stats"]["n_aug"] == aug["n"]
        for k in ("winner", "sigma"):
            np.testing.assert_array_equal(to_np(out[k]), ref[k])
        np.testing.assert_array_equal(to_np(out["tau"]), ref["tau_orig"])
        for k in ("n_major", "n_valuations", "n_odd_switches",
                  "n_even_switches"):
            assert out["stats"][k] == ref[k], k

"""Rows of hundreds to thousands of entries, decided by a whole block
(csrc/pg_coarse.h), around the lines where a thread takes them instead, for
either player, with random keys and with many that tie; single games in
either form of All_Odd and batches, against the oracle, exactly."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import orc
from paper_1705_02313_amd import synth
from paper_1705_02313_amd.pg import Batch, Game
from tests.helpers import to_np
from tests.test_gpu_batch import _check, _drain

pytestmark = pytest.mark.gpu


def _game(kind, n, rows, degree, owner, seed):
    """A random game or a chain whose priorities rise by stairs (most of its
    vertices share a few roots), with `rows` scattered vertices of `owner`
    leading to `degree` more targets each, some of them repeated."""
    rng = np.random.default_rng([n, rows, degree, seed])
    if kind == "stairs":
        g = synth.chain_game(n, seed)
        pri = np.arange(n, dtype=np.int32)
        for a in range(0, n, 700):
            rng.shuffle(pri[a:a + 700])
        g["pri"] = pri
    else:
        g = synth.random_game(n, 2, 5, seed)
    who = rng.choice(n, rows, replace=False)
    g["owner"][who] = owner
    src = np.concatenate([np.repeat(np.arange(n), np.diff(g["offsets"])),
                          np.repeat(who, degree)])
    tgt = np.concatenate([g["targets"], rng.integers(0, n, rows * degree)])
    if kind == "stairs":   # half of them near the row's owner
        k = rows * degree // 2
        tgt[-k:] = (src[-k:] + rng.integers(1, 900, k)) % n
    order = np.argsort(src, kind="stable")
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum(np.bincount(src, minlength=n))
    return dict(g, m=int(off[-1]), offsets=off,
                targets=tgt[order].astype(np.int32))


@pytest.mark.parametrize("owner", [0, 1], ids=["even", "odd"])
@pytest.mark.parametrize("kind", ["random", "stairs"])
@pytest.mark.parametrize("n,rows,degree", [
    (9000, 1, 127), (9000, 3, 125), (9000, 40, 150), (9000, 9, 2500),
    (9000, 1200, 300), (40009, 4, 9000), (140003, 3, 20000),
    (140003, 700, 260)])
def test_wide_rows(n, rows, degree, kind, owner):
    g = _game(kind, n, rows, degree, owner, 7)
    ref = orc.solve(g)
    for switch in ("rows", "buckets"):
        with Game.from_dict(g, switch=switch) as d:
            out = d.solve()
            for k in ("winner", "sigma"):
                np.testing.assert_array_equal(to_np(out[k]), ref[k])
            np.testing.assert_array_equal(to_np(out["tau"]), ref["tau_orig"])
            for k in ("n_major", "n_valuations", "n_odd_switches",
                      "n_even_switches"):
                assert out["stats"][k] == ref[k], k


def test_wide_rows_in_a_batch():
    games = [_game(kind, 7000, rows, degree, owner, 3)
             for kind in ("random", "stairs") for owner in (0, 1)
             for rows, degree in ((1, 127), (5, 400), (500, 200), (3, 6000))]
    with Batch(max_vertices=1 << 18, max_edges=1 << 21) as b:
        out = _drain(b, [b.submit(g) for g in games])
    for g, t in zip(games, sorted(out)):
        _check(g, out[t])

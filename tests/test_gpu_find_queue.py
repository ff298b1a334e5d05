"""The changed part found over hubs of some hundreds to 2,048 in-edges, whose
sources all play through them: past a block's LDS lists every wave takes
chunks of the queue for the few sources it has just found, which fits the
queue in the wide games here and asks for more than it holds in the others
(the step then gives up and a full valuation follows).  Against the oracle,
exactly."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import orc
from paper_1705_02313_amd import synth
from paper_1705_02313_amd.pg import Game
from tests.helpers import to_np

pytestmark = pytest.mark.gpu


def _hubs(n, hubs, degree, few):
    """One Odd vertex 0 that prefers its second successor, `hubs` Odd vertices
    on it, `degree` Odd vertices on each of those, and the rest (Odd) on
    scattered Even ones: the first All_Odd switches vertex 0 alone, and with
    it the play of every hub and source changes."""
    rng = np.random.default_rng([n, hubs, degree])
    sources = hubs * degree
    first = 1 + hubs + sources          # the Even vertices and the rest
    evens = 2 + (n - first - 2) // 50
    assert first + evens <= n
    owner = np.ones(n, np.uint8)
    owner[first:first + evens] = 0
    a, b = first, first + 1
    row = np.empty(n, np.int64)         # the only target, but vertex 0's
    row[1:1 + hubs] = 0
    row[1 + hubs:first] = 1 + np.arange(sources) // degree
    row[first:first + evens] = 1 + rng.integers(0, hubs, evens)
    row[first + evens:] = first + 2 + rng.integers(0, max(evens - 2, 1),
                                                   n - first - evens)
    tgt = np.concatenate([[a, b], row[1:]]).astype(np.int32)
    off = np.arange(n + 1, dtype=np.int64) + 1
    off[0] = 0
    if few:
        pri = rng.integers(0, 3, n).astype(np.int32)
        pri[a], pri[b] = 4, 5
    else:
        top = n + (n & 1)
        pri = rng.permutation(n).astype(np.int32)
        pri[a], pri[b] = top, top + 1
    return {"n": n, "m": int(off[-1]), "offsets": off, "targets": tgt,
            "owner": owner, "pri": pri}


@pytest.mark.parametrize("few", [False, True], ids=["ranks", "counts"])
@pytest.mark.parametrize("n,hubs,degree", [
    (6500, 3, 1500),        # more chunks than places
    (7000, 2, 2048),
    (17000, 8, 2040),
    (150000, 64, 2040),
    (60000, 3, 1500),       # fits
    (60000, 24, 300),
    (200000, 2, 2048)])
def test_hubs_within_the_degree_bound(n, hubs, degree, few):
    g = _hubs(n, hubs, degree, few)
    ref = orc.dense_solve(g) if few else orc.solve(g)
    with Game.from_dict(g) as d:
        for profiled in (False, True):
            d.profile(profiled)
            out = d.solve()
            for k in ("winner", "sigma"):
                np.testing.assert_array_equal(to_np(out[k]), ref[k])
            np.testing.assert_array_equal(to_np(out["tau"]), ref["tau_orig"])
            for k in ("n_major", "n_valuations"):
                assert out["stats"][k] == ref[k], k
        ran = d.profile_read()
        assert "inc_block" in ran
        if hubs * (degree + 1) >= 4096:
            assert "inc_find" in ran


def test_a_hub_beyond_the_degree_bound_costs_no_ranks():
    """A find that gives up at a hub leaves the full valuations that follow on
    coarse keys: nothing of the run sorts or ranks."""
    g = _hubs(20000, 3, 3000, False)
    ref = orc.solve(g)
    with Game.from_dict(g) as d:
        d.profile()
        out = d.solve()
        ran = d.profile_read()
    np.testing.assert_array_equal(to_np(out["sigma"]), ref["sigma"])
    assert out["stats"]["n_valuations"] == ref["n_valuations"]
    assert "inc_find" in ran or "inc_block" in ran
    assert not {"sort_split", "sort_pass", "lr_sum1", "lr_emit1"} & set(ran)


@pytest.mark.parametrize("few", [0, 4], ids=["ranks", "counts"])
@pytest.mark.parametrize("n,hubs,degree", [
    (9000, 30, 126), (9000, 60, 140), (9000, 3, 2000), (60000, 40, 1200),
    (60000, 400, 129), (140003, 60, 2047), (140003, 60, 2100)])
def test_random_games_with_hubs(n, hubs, degree, few):
    """Random games whose hubs change their plays all along a run, with some
    edges into them repeated."""
    rng = np.random.default_rng([n, hubs, degree])
    g = synth.few_priorities_game(n, 2, 4, few, 3) if few else \
        synth.random_game(n, 2, 4, 3)
    src = np.concatenate([np.repeat(np.arange(n), np.diff(g["offsets"])),
                          rng.integers(0, n, hubs * degree)])
    tgt = np.concatenate([g["targets"],
                          np.repeat(rng.choice(n, hubs, replace=False),
                                    degree)])
    again = rng.random(src.size) < 0.1
    src, tgt = np.append(src, src[again]), np.append(tgt, tgt[again])
    order = np.lexsort((rng.random(src.size), src))
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum(np.bincount(src, minlength=n))
    g = dict(g, m=int(off[-1]), offsets=off,
             targets=tgt[order].astype(np.int32))
    ref = orc.dense_solve(g) if few else orc.solve(g)
    with Game.from_dict(g) as d:
        for _ in range(2):
            out = d.solve()
            for k in ("winner", "sigma"):
                np.testing.assert_array_equal(to_np(out[k]), ref[k])
            np.testing.assert_array_equal(to_np(out["tau"]), ref["tau_orig"])
            for k in ("n_major", "n_valuations"):
                assert out["stats"][k] == ref[k], k

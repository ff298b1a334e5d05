"""Strategies that name vertices outside their rows, in games above the
one-block size: the choice is kept where it beats the row, and is followed
when its target's play changes in a later step of a few switches.  Best
responses against the oracle's, solves against the same solves on full
valuations (a trace asks for those)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import orc
from paper_1705_02313_amd import synth
from paper_1705_02313_amd.pg import PG_EINADMISSIBLE, Game, PgError
from tests.helpers import to_np

pytestmark = pytest.mark.gpu

HUBS, DEGREE, CHOOSERS = 3, 400, 300


def _game(n, few, wide):
    """Odd's vertex 0 prefers b to a and many others play through it.
    CHOOSERS Odd vertices (rows of `wide` entries) and as many followers that
    would rather join them than play to f once vertex 0 has switched (a, f
    and b have large odd priorities, in that order); the strategy of the test
    lets each chooser name a vertex that plays through 0."""
    rng = np.random.default_rng([n, wide])
    src = 1 + HUBS
    cho = src + HUBS * DEGREE
    fol = cho + CHOOSERS
    a, b, f = range(fol + CHOOSERS, fol + CHOOSERS + 3)
    owner = np.ones(n, np.uint8)
    owner[a:] = 0
    rows = [[a, b]] + [[0]] * HUBS
    rows += [[1 + i // DEGREE] for i in range(HUBS * DEGREE)]
    rows += [list(rng.integers(f + 1, n, wide)) for _ in range(CHOOSERS)]
    rows += [[f, cho + i] for i in range(CHOOSERS)]
    rows += [[int(rng.integers(a, n))] for _ in range(a, n)]
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum([len(r) for r in rows])
    pri = rng.integers(0, 4, n) if few else rng.permutation(n)
    top = 4 if few else n + (n & 1)
    pri[a], pri[f], pri[b] = top + 1, top + 3, top + 5
    g = {"n": n, "m": int(off[-1]), "offsets": off,
         "targets": np.concatenate(rows).astype(np.int32), "owner": owner,
         "pri": pri.astype(np.int32)}
    return g, np.arange(cho, fol), np.arange(src, src + CHOOSERS)


def _oracle_best_response(aug, sigma, tau, few):
    by_pri = None if few else orc.order_by_pri(aug["pri"])
    t, nval = tau.copy(), 0
    while True:
        succ = np.where(aug["owner"] == 1, t, sigma).astype(np.int32)
        nval += 1
        if few:
            counts, top, values, rc = orc.dense_valuation(succ, aug["pri"])
            assert rc == 0
            key = None
            t, c = orc.dense_odd_switch(aug, counts, top, values, t)
        else:
            key, _, rc = orc.valuation(succ, aug["pri"], by_pri=by_pri)
            assert rc == 0
            t, c = orc.odd_switch(aug, key, t)
        if c == 0:
            return t, key, nval


def _solve(d, **kw):
    try:
        return d.solve(keep_dummies=True, **kw)
    except PgError as e:
        assert e.status == PG_EINADMISSIBLE
        return None


def _same_solve(d, **start):
    a, b = _solve(d, **start), _solve(d, trace=4096, **start)
    if b is None:   # (direct edges can close a cycle that the dummies cut)
        assert a is None
        return
    for k in ("winner", "sigma", "tau"):
        np.testing.assert_array_equal(to_np(a[k]), to_np(b[k]))
    for k in ("n_major", "n_valuations", "n_odd_switches",
              "n_even_switches"):
        assert a["stats"][k] == b["stats"][k], k


@pytest.mark.parametrize("few", [False, True], ids=["ranks", "counts"])
@pytest.mark.parametrize("switch", ["rows", "buckets"])
@pytest.mark.parametrize("wide", [1, 5, 128, 129, 700])
def test_choices_outside_rows_are_followed(few, switch, wide):
    g, who, to = _game(40001, few, wide)
    aug = orc.dense_preprocess(g) if few else orc.preprocess(g)
    assert aug["n"] == g["n"]
    with Game.from_dict(g, switch=switch) as d:
        sigma, tau = d.initial_strategies()
        tau[who] = to
        want = _oracle_best_response(aug, sigma, tau, few)
        assert (want[0][who] == to).all() and want[2] == 3
        for _ in range(2):
            got = d.best_response(sigma, tau)
            np.testing.assert_array_equal(got[0], want[0])
            if not few:
                np.testing.assert_array_equal(got[1], want[1])
            assert got[2] == want[2]
            _same_solve(d, init_sigma=sigma, init_tau=tau)
        # an Even choice outside its row
        sigma[g["n"] - 1] = to[0]
        _same_solve(d, init_sigma=sigma, init_tau=tau)
        # all in their rows again
        out = d.solve()
    ref = orc.dense_solve(g) if few else orc.solve(g)
    np.testing.assert_array_equal(to_np(out["sigma"]), ref["sigma"])
    assert out["stats"]["n_valuations"] == ref["n_valuations"]


@pytest.mark.parametrize("few", [0, 4])
@pytest.mark.parametrize("n,seed", [(20011, 4), (60000, 7)])
def test_a_reported_tau_as_a_start(n, seed, few):
    """The tau a solve reports names the dummies' targets: no edges of the
    modified game.  A tenth of its choices, the others as they were."""
    g = synth.few_priorities_game(n, 2, 8, few, seed) if few else \
        synth.random_game(n, 2, 8, seed)
    rng = np.random.default_rng(seed)
    with Game.from_dict(g) as d:
        assert d.n_aug > d.n
        tau = d.solve()["tau"]
        inner = d.solve(keep_dummies=True)["tau"]
        tau = np.where(rng.random(d.n_aug) < 0.1, tau, inner)
        assert (tau != inner).sum() > 100
        _same_solve(d, init_tau=tau)
        sigma = d.solve(max_major=3, checkpoint=True)["sigma"]
        _same_solve(d, init_sigma=sigma, init_tau=tau)

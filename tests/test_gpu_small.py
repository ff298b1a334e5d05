"""Games solved and valued whole in one block (csrc/pg_small.hip) against the
oracle: one vertex up to the first sizes that take the general path again (by
vertices and by edges), ng chains at and beyond the block's bound, SI-Reset,
caps, warm starts and inadmissible strategies.  Everything is exact.
"""
from __future__ import annotations

import numpy as np
import pytest

from oracle import orc
from paper_1705_02313_amd import synth
from paper_1705_02313_amd.pg import (PG_BR_SI_RESET, PG_EINADMISSIBLE,
                                     PG_EINVAL, Game, PgError, solve_noalloc)
from tests.helpers import oracle_trajectory, to_np

pytestmark = pytest.mark.gpu

COUNTS = ("n_major", "n_valuations", "n_odd_switches", "n_even_switches")


def _same(out, ref):
    for k in ("winner", "sigma"):
        np.testing.assert_array_equal(to_np(out[k]), ref[k])
    np.testing.assert_array_equal(to_np(out["tau"]), ref["tau_orig"])
    for k in COUNTS:
        assert out["stats"][k] == ref[k], k


def _path_game(n):
    """One play through every vertex with priorities rising along it: an ng
    chain of n vertices (every vertex Odd but the last, which may stop)."""
    off = np.arange(n + 1, dtype=np.int64)
    tgt = np.append(np.arange(1, n), 0).astype(np.int32)
    owner = np.ones(n, np.uint8)
    owner[n - 1] = 0
    return {"n": n, "m": n, "offsets": off, "targets": tgt, "owner": owner,
            "pri": np.arange(n, dtype=np.int32)}


def _self_loop():
    return {"n": 1, "m": 1, "offsets": np.array([0, 1], np.int64),
            "targets": np.zeros(1, np.int32), "owner": np.zeros(1, np.uint8),
            "pri": np.zeros(1, np.int32)}


SIZES = [(2, 1, 1), (3, 2, 2), (63, 2, 4), (770, 2, 5), (1024, 2, 5),
         (1536, 1, 3), (3000, 2, 10), (4600, 2, 5), (4700, 2, 5),
         (4500, 8, 16)]


@pytest.mark.parametrize("n,dmin,dmax", SIZES)
@pytest.mark.parametrize("device", [False, True])
def test_solves(n, dmin, dmax, device):
    g = synth.random_game(n, dmin, dmax, n)
    with Game.from_dict(g, device=device) as d:
        aug, ex = orc.preprocess(g), d.export()
        for k in ("offsets", "targets", "owner", "pri"):
            np.testing.assert_array_equal(ex[k], aug[k])
        _same(d.solve(), orc.solve(g))
        _same(d.solve(best_response=PG_BR_SI_RESET), orc.solve(g, reset=True))
    _same(solve_noalloc(g, device=device), orc.solve(g))


@pytest.mark.parametrize("n", [2, 63, 770, 1500, 4600])
@pytest.mark.parametrize("device", [False, True])
def test_valuations_along_a_run(n, device):
    g = synth.random_game(n, 1, 5, n + 1)
    aug = orc.preprocess(g)
    with Game.from_dict(g, device=device) as d:
        for sigma, tau, key in oracle_trajectory(aug, 12):
            k, f = d.valuation(sigma, tau)
            np.testing.assert_array_equal(to_np(k), key)
            assert f == int((key != orc.KEY_TOP).sum())


@pytest.mark.parametrize("n", [1, 2, 254, 256, 257, 258, 300, 3000])
def test_long_ng_chains(n):
    g = _path_game(n) if n > 1 else _self_loop()
    with Game.from_dict(g) as d:
        _same(d.solve(), orc.solve(g))
        aug = orc.preprocess(g)
        sigma, tau = orc.initial_strategies(aug)
        succ = np.where(aug["owner"] == 1, tau, sigma).astype(np.int32)
        key, nf, rc = orc.valuation(succ, aug["pri"])
        assert rc == 0
        k, f = d.valuation(sigma, tau)
        np.testing.assert_array_equal(to_np(k), key)
        assert f == nf


def test_best_responses_and_caps():
    g = synth.random_game(1800, 2, 6, 12)
    with Game.from_dict(g) as d:
        whole = d.solve()
        for cap in [{"max_major": k} for k in
                    range(1, whole["stats"]["n_major"])] + \
                [{"max_inner": k} for k in (1, 2, 3)]:
            a = d.solve(checkpoint=True, keep_dummies=True, **cap)
            b = d.solve(checkpoint=True, keep_dummies=True, trace=4096, **cap)
            assert a.get("stopped") == b.get("stopped"), cap
            for k in ("sigma", "tau"):
                np.testing.assert_array_equal(to_np(a[k]), to_np(b[k]))
            for k in COUNTS:
                assert a["stats"][k] == b["stats"][k], (cap, k)
            tau, key, _ = d.best_response(a["sigma"], a["tau"])
            with Game.from_dict(g, switch="rows") as e:
                tau2, key2, _ = e.best_response(a["sigma"], a["tau"])
            np.testing.assert_array_equal(to_np(tau), to_np(tau2))
            np.testing.assert_array_equal(to_np(key), to_np(key2))


def test_loads_refused_or_left_to_the_general_path():
    g = synth.random_game(50, 2, 4, 5)
    for k, i, x in (("targets", 7, 50), ("owner", 3, 2), ("pri", 9, -1),
                    ("offsets", 4, 0), ("pri", 0, 2**31 - 1)):
        h = {q: np.array(a) for q, a in g.items()}
        h[k][i] = x
        with pytest.raises(PgError) as e:
            Game.from_dict(h)
        assert e.value.status == PG_EINVAL
    h = dict(g, pri=g["pri"] // 2 * 2)   # repeated: count valuations
    with Game.from_dict(h) as d:
        assert d.d > 0
        d.solve()


def test_refused_strategies():
    g = synth.random_game(40, 2, 4, 3)
    with Game.from_dict(g) as d:
        sigma, tau = d.initial_strategies()
        bad = np.array(tau)
        bad[int(np.flatnonzero(g["owner"] == 1)[0])] = d.n_aug
        with pytest.raises(PgError) as e:
            d.valuation(sigma, bad)
        assert e.value.status == PG_EINVAL
    # two vertices of Even circling with an odd largest priority
    g = {"n": 2, "m": 2, "offsets": np.array([0, 1, 2], np.int64),
         "targets": np.array([1, 0], np.int32),
         "owner": np.zeros(2, np.uint8), "pri": np.array([2, 3], np.int32)}
    with Game.from_dict(g, preprocess=False) as d:
        s = np.array([1, 0], np.int32)
        t = np.full(2, -1, np.int32)
        for call in (d.valuation, d.best_response):
            with pytest.raises(PgError) as e:
                call(s, t)
            assert e.value.status == PG_EINADMISSIBLE
        with pytest.raises(PgError) as e:
            d.solve(init_sigma=s)
        assert e.value.status == PG_EINADMISSIBLE

"""A handle after a refused strategy: runs that an inadmissible sigma stops in
a valuation by the changed part (the odd cycle closes when Odd answers), and
then the runs that follow on the same handle, against the oracle."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

from oracle import orc
from paper_1705_02313_amd.pg import (PG_EINADMISSIBLE, Game, PgError,
                                     SolveOpts, Stats, lib)
from tests.helpers import to_np

pytestmark = pytest.mark.gpu

HUBS, DEGREE, CHOOSERS = 3, 400, 300


def _game(n, few):
    """Odd's vertex 0 prefers b to a; HUBS Odd vertices lead to it, DEGREE
    to each of those, and CHOOSERS Odd vertices would rather join them once
    vertex 0 has switched.  The last two vertices: an Even one of odd
    priority and an Odd one that prefers it, so a sigma that answers with
    the Odd one closes an odd cycle in the step after the first All_Odd."""
    rng = np.random.default_rng(n)
    src = 1 + HUBS
    cho = src + HUBS * DEGREE
    a, b = cho + CHOOSERS, cho + CHOOSERS + 1
    e, o = n - 2, n - 1
    owner = np.ones(n, np.uint8)
    owner[a:e + 1] = 0
    rows = [[a, b]] + [[0]] * HUBS
    rows += [[1 + i // DEGREE] for i in range(HUBS * DEGREE)]
    rows += [[int(rng.integers(b + 1, e)), src + i] for i in range(CHOOSERS)]
    rows += [[int(rng.integers(a, e))] for _ in range(a, e)]
    rows += [[o], [b + 1, e]]
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum([len(r) for r in rows])
    pri = rng.integers(0, 4, n) if few else rng.permutation(n)
    top = 4 if few else n + (n & 1)
    pri[a], pri[b], pri[e] = top, top + 1, top + 3
    g = {"n": n, "m": int(off[-1]), "offsets": off,
         "targets": np.concatenate(rows).astype(np.int32), "owner": owner,
         "pri": pri.astype(np.int32)}
    return g, e, o


@pytest.mark.parametrize("few", [False, True], ids=["ranks", "counts"])
def test_runs_after_a_refused_strategy(few):
    g, e, o = _game(9001, few)
    ref = orc.dense_solve(g) if few else orc.solve(g)
    with Game.from_dict(g) as d:
        assert d.n_aug == g["n"]
        sigma, tau = d.initial_strategies()
        bad = sigma.copy()
        bad[e] = o
        with Game.from_dict(g) as fresh:
            want = fresh.best_response(sigma, tau)
        for again in range(2):
            with pytest.raises(PgError) as err:
                if again:
                    d.best_response(bad, tau)
                else:
                    d.solve(init_sigma=bad)
            assert err.value.status == PG_EINADMISSIBLE
            got = d.best_response(sigma, tau)
            np.testing.assert_array_equal(got[0], want[0])
            if not few:
                np.testing.assert_array_equal(got[1], want[1])
                np.testing.assert_array_equal(
                    got[1], d.valuation(sigma, got[0])[0])
            assert got[2] == want[2]
            with pytest.raises(PgError) as err:
                d.solve(init_sigma=bad)
            assert err.value.status == PG_EINADMISSIBLE
            out = d.solve()
            for k in ("winner", "sigma"):
                np.testing.assert_array_equal(to_np(out[k]), ref[k])
            np.testing.assert_array_equal(to_np(out["tau"]), ref["tau_orig"])
            for k in ("n_major", "n_valuations"):
                assert out["stats"][k] == ref[k], k


@pytest.mark.parametrize("few", [False, True], ids=["ranks", "counts"])
@pytest.mark.parametrize("n", [3001, 9001])   # in one block, and above
def test_counts_of_a_refused_run(n, few):
    """What a refused run had done is reported whatever form it took: as by
    the same run on full valuations (a trace asks for those)."""
    g, e, o = _game(n, few)
    winner = np.zeros(n, np.uint8)
    with Game.from_dict(g) as d:
        bad, tau = d.initial_strategies()
        bad[e] = o
        seen = []
        for cap in (0, 64):
            finite = np.zeros(64, np.int64)
            opts = SolveOpts(0, 0, 0, 0, bad.ctypes.data, tau.ctypes.data,
                             cap, 0, None, finite.ctypes.data, None, None)
            st = Stats()
            rc = lib().pg_solve(d._h, ctypes.byref(opts),
                                winner.ctypes.data, None, None,
                                ctypes.byref(st), None)
            assert rc == PG_EINADMISSIBLE
            seen.append([st.n_major, st.n_valuations, st.n_odd_switches,
                         st.n_even_switches])
        assert seen[0] == seen[1]
        nv = ctypes.c_int32(-1)
        rc = lib().pg_best_response(d._h, bad.ctypes.data, tau.ctypes.data,
                                    None, ctypes.byref(nv), 0, 0, None)
        assert rc == PG_EINADMISSIBLE and nv.value == seen[1][1]

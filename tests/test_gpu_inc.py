"""Valuations by their changed part (csrc/pg_inc.hip) against the oracle, at
the sizes and shapes where the path changes: games that always fit one block
and the first that do not, hubs beyond the in-degree bound, repeated edges,
ng chains beyond the comparison's bound, games whose vertices share a few
roots (their coarse keys tie); and runs stopped by caps against the
same runs on full valuations (a trace asks for those).  Everything is exact.
"""
from __future__ import annotations

import numpy as np
import pytest

from oracle import orc
from paper_1705_02313_amd import synth
from paper_1705_02313_amd.pg import Batch, Game
from tests.helpers import to_np
from tests.test_gpu_batch import _check, _drain

pytestmark = pytest.mark.gpu


def _csr(rows, owner, pri):
    off = np.zeros(len(rows) + 1, np.int64)
    off[1:] = np.cumsum([len(r) for r in rows])
    return {"n": len(rows), "m": int(off[-1]), "offsets": off,
            "targets": np.concatenate(rows).astype(np.int32),
            "owner": np.asarray(owner, np.uint8),
            "pri": np.asarray(pri, np.int32)}


def _rows(g):
    return np.split(g["targets"], g["offsets"][1:-1])


def _hub(n, seed):
    """Every third vertex also leads to vertex 0."""
    g = synth.random_game(n, 2, 4, seed)
    rows = [np.append(r, 0) if v % 3 == 1 else r
            for v, r in enumerate(_rows(g))]
    return _csr(rows, g["owner"], g["pri"])


def _doubled(n, seed):
    g = synth.random_game(n, 2, 4, seed)
    return _csr([np.repeat(r, 2) for r in _rows(g)], g["owner"], g["pri"])


def _rising(n, seed):
    """A chain whose priorities rise along it: ng chains as long as plays."""
    g = synth.chain_game(n, seed)
    g["pri"] = np.arange(n, dtype=np.int32)
    return g


def _stairs(n, seed, step):
    """A chain whose priorities rise by stairs of `step` vertices: most
    vertices share a few roots and the ng chains have about n / step links."""
    g = synth.chain_game(n, seed)
    rng = np.random.default_rng(seed)
    pri = np.arange(n, dtype=np.int32)
    for a in range(0, n, step):
        rng.shuffle(pri[a:a + step])
    g["pri"] = pri
    return g


GAMES = {
    "tiny": lambda: synth.random_game(3, 2, 2, 1),
    "one_block": lambda: synth.random_game(900, 2, 5, 2),
    "block_edge_below": lambda: synth.random_game(3050, 2, 5, 3),
    "block_edge_above": lambda: synth.random_game(3150, 2, 5, 3),
    "mid": lambda: synth.random_game(20011, 2, 8, 4),
    "large": lambda: synth.random_game(150001, 2, 5, 5),
    "large_hub": lambda: _hub(140003, 14),
    "chain": lambda: synth.chain_game(60013, 6),
    "hub": lambda: _hub(20000, 7),
    "doubled": lambda: _doubled(6001, 8),
    "doubled_small": lambda: _doubled(701, 9),
    "rising": lambda: _rising(3000, 10),
    "rising_large": lambda: _rising(12001, 11),
    "stairs": lambda: _stairs(40009, 12, 600),
    "stairs_wide": lambda: _stairs(40009, 13, 8000),
}


@pytest.mark.parametrize("name", sorted(GAMES))
@pytest.mark.parametrize("switch", ["rows", "buckets"])
def test_runs_equal_the_oracle(name, switch):
    g = GAMES[name]()
    ref = orc.solve(g)
    with Game.from_dict(g, switch=switch) as d:
        for _ in range(2):   # the in-edge lists and epochs live on
            out = d.solve()
            for k in ("winner", "sigma"):
                np.testing.assert_array_equal(to_np(out[k]), ref[k])
            np.testing.assert_array_equal(to_np(out["tau"]), ref["tau_orig"])
            for k in ("n_major", "n_valuations", "n_odd_switches",
                      "n_even_switches"):
                assert out["stats"][k] == ref[k], k
        # a best response ends with the ranks of every vertex
        sigma, tau = d.initial_strategies()
        tau, key, _ = d.best_response(ref["sigma"], tau)
        k2, _ = d.valuation(ref["sigma"], tau)
        np.testing.assert_array_equal(to_np(key), to_np(k2))


@pytest.mark.parametrize("d", [2, 4, 6, 12, 27])
@pytest.mark.parametrize("name", ["one_block", "mid", "chain", "hub",
                                  "doubled"])
def test_count_runs_equal_the_oracle(name, d):
    g = GAMES[name]()
    rng = np.random.default_rng(d)
    g["pri"] = rng.integers(0, d, g["n"]).astype(np.int32)
    ref = orc.dense_solve(g)
    with Game.from_dict(g) as h:
        for _ in range(2):
            out = h.solve()
            for k in ("winner", "sigma"):
                np.testing.assert_array_equal(to_np(out[k]), ref[k])
            np.testing.assert_array_equal(to_np(out["tau"]), ref["tau_orig"])
            for k in ("n_major", "n_valuations"):
                assert out["stats"][k] == ref[k], k


@pytest.mark.parametrize("name", ["one_block", "mid", "chain"])
def test_caps_stop_at_the_same_strategies(name):
    g = GAMES[name]()
    with Game.from_dict(g) as d:
        whole = d.solve()
        majors = whole["stats"]["n_major"]
        caps = [{"max_major": k} for k in range(1, majors)] + \
            [{"max_inner": k} for k in (1, 2, 3, 4)]
        for cap in caps:
            a = d.solve(checkpoint=True, keep_dummies=True, **cap)
            b = d.solve(checkpoint=True, keep_dummies=True, trace=4096, **cap)
            assert a.get("stopped") == b.get("stopped"), cap
            for k in ("sigma", "tau"):
                np.testing.assert_array_equal(to_np(a[k]), to_np(b[k]))
            for k in ("n_major", "n_valuations", "n_odd_switches",
                      "n_even_switches"):
                assert a["stats"][k] == b["stats"][k], (cap, k)


@pytest.mark.parametrize("names", [
    ("stairs", "stairs_wide", "hub", "doubled", "chain", "tiny", "mid"),
    ("rising", "mid", "stairs_wide"),   # chains too long: ranks in a layout
])
def test_batches_equal_the_oracle(names):
    games = [GAMES[k]() for k in names]
    with Batch(max_vertices=1 << 18, max_edges=1 << 20) as b:
        tickets = [b.submit(g) for g in games]
        out = _drain(b, list(tickets))
    for g, t in zip(games, tickets):
        _check(g, out[t])

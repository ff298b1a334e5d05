"""The library over a HIP runtime that refuses memory: tests/runtime_main.c,
a program with a hipMalloc and a hipHostMalloc of its own, run as a child."""
from __future__ import annotations

import os
import subprocess

import numpy as np
import pytest

from oracle import orc
from paper_1705_02313_amd import pg, synth

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = "/opt/rocm/lib"


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("rt") / "runtime_main")
    libdir = os.path.dirname(pg.LIB_PATH)
    subprocess.run(["gcc", "-std=gnu99", "-O1", "-Wall", "-rdynamic",
                    os.path.join(HERE, "runtime_main.c"), "-o", out,
                    pg.LIB_PATH, "-L" + ROCM, "-lamdhip64", "-ldl",
                    "-Wl,--disable-new-dtags", "-Wl,-rpath," + libdir,
                    "-Wl,-rpath," + ROCM], check=True)

    def go(*args):
        r = subprocess.run([out, *map(str, args)], capture_output=True,
                           text=True, timeout=100)
        assert r.returncode == 0, (r.returncode, r.stdout, r.stderr[-2000:])
        return [ln.split()[1:] for ln in r.stdout.splitlines()
                if ln.split()[:1] == [args[0]]]
    return go


def _write(path, g):
    with open(path, "wb") as f:
        np.array([g["n"], g["m"]], np.int64).tofile(f)
        np.asarray(g["offsets"], np.int64).tofile(f)
        np.asarray(g["targets"], np.int32).tofile(f)
        np.asarray(g["owner"], np.uint8).tofile(f)
        np.asarray(g["pri"], np.int32).tofile(f)
    return path


def _with_rising_path(g, length):
    """g and a path of Odd vertices into it whose priorities rise above all
    others: nearest-greater chains of `length` links."""
    n, m = g["n"], g["m"]
    into = int(np.flatnonzero(g["owner"] == 0)[0])
    return {"n": n + length, "m": m + length,
            "offsets": np.append(g["offsets"], m + 1 + np.arange(length)),
            "targets": np.append(g["targets"],
                                 [*range(n + 1, n + length), into]),
            "owner": np.append(g["owner"], np.ones(length, np.uint8)),
            "pri": np.append(g["pri"], n + np.arange(length))}


def test_counts_of_a_run_that_finds_no_memory_on_the_way(run, tmp_path):
    """A small game's run that turns to the general path, which finds no
    memory for its in-edges: the counts and the cap go on."""
    g = _with_rising_path(synth.random_game(2000, 2, 5, 10), 600)
    ref = orc.solve(g)
    assert ref["n_major"] > 3
    whole, capped = run("deep", _write(tmp_path / "g", g))
    assert [int(x) for x in whole] == [pg.PG_OK, ref["n_major"],
                                       ref["n_valuations"]]
    assert [int(x) for x in capped[:2]] == [pg.PG_EITERLIMIT, 2]


def test_a_refused_run_keeps_no_scratch(run, tmp_path):
    """The in-edges of a large game are built over pairs of 8 bytes an edge,
    which a run gives back also when its first valuation is refused."""
    g = synth.random_game(140001, 2, 5, 3)
    n, m = g["n"], g["m"]
    g = {"n": n + 2, "m": m + 2,
         "offsets": np.append(g["offsets"], [m + 1, m + 2]),
         "targets": np.append(g["targets"], [n + 1, n]),
         "owner": np.append(g["owner"], [0, 1]),
         "pri": np.append(g["pri"], [n + n % 2 + 1, n + n % 2])}
    refused, fine = run("pairs", _write(tmp_path / "g", g))
    assert int(refused[0]) == pg.PG_EINADMISSIBLE
    assert int(fine[0]) == pg.PG_OK
    assert int(refused[1]) == int(fine[1])


def test_memory_kept_for_the_next_batch_is_given_up(run, tmp_path):
    """What a freed batch left for the next one goes back when a load finds
    no other memory; an arena that fits only in its exact size is made so."""
    g = synth.random_game(200000, 2, 5, 3)
    assert int(run("idle", _write(tmp_path / "g", g))[0][0]) == pg.PG_OK
    assert int(run("exact")[0][0]) == pg.PG_OK


def test_errors_of_other_calls_are_not_taken_over(run, tmp_path):
    """The error that a HIP call of the program left behind is not this
    library's: a small load and a poll of several games go through."""
    g = synth.random_game(1000, 2, 5, 3)
    got = run("stale", _write(tmp_path / "g", g))
    assert [int(x[0]) for x in got] == [pg.PG_OK, pg.PG_OK]

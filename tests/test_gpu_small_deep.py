"""Valuations and best responses of small games whose nearest-greater chains
are too deep for the one-block form: the general path's results each time, and
the one-block form is tried less and less often."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import orc
from paper_1705_02313_amd import synth
from paper_1705_02313_amd.pg import Game
from tests.helpers import to_np
from tests.test_gpu_off_row import _oracle_best_response
from tests.test_gpu_runtime import _with_rising_path

pytestmark = pytest.mark.gpu


def test_deep_valuations_are_not_tried_twice_each_time():
    g = _with_rising_path(synth.random_game(2000, 2, 5, 10), 600)
    aug = orc.preprocess(g)
    sigma, tau = orc.initial_strategies(aug)
    succ = np.where(aug["owner"] == 1, tau, sigma).astype(np.int32)
    key, nf, rc = orc.valuation(succ, aug["pri"])
    assert rc == 0
    br = _oracle_best_response(aug, sigma, tau, False)
    with Game.from_dict(g) as d:
        d.profile()
        for _ in range(20):
            got, n = d.valuation(sigma, tau)
            np.testing.assert_array_equal(to_np(got), key)
        assert d.profile_read()["small"]["calls"] <= 5
        for _ in range(3):
            t, k, nv = d.best_response(sigma, tau)
            np.testing.assert_array_equal(to_np(t), br[0])
            np.testing.assert_array_equal(to_np(k), br[1])
            assert nv == br[2]

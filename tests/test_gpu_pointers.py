"""Device buffers that are not what a kernel would read or write in place:
elements off their boundaries, and pinned host memory given as device
pointers.  They are copied; results against the oracle, exactly."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

from oracle import orc
from paper_1705_02313_amd import synth
from paper_1705_02313_amd.pg import (PG_KEEP_DUMMIES, PG_OFFSETS_I32, PG_OK,
                                     PG_PTR_DEVICE, Batch, SolveOpts,
                                     Stats, lib)
from tests.helpers import to_np

pytestmark = pytest.mark.gpu


def _place(a, where, shift):
    """The array's bytes in device or pinned memory, `shift` bytes in."""
    raw = torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).copy())
    if where == "device":
        buf = torch.zeros(raw.numel() + 16, dtype=torch.uint8, device="cuda")
    else:
        buf = torch.zeros(raw.numel() + 16, dtype=torch.uint8,
                          pin_memory=True)
    buf[shift:shift + raw.numel()] = raw
    return buf, buf.data_ptr() + shift


@pytest.mark.parametrize("where,shift", [("device", 0), ("device", 1),
                                         ("device", 4), ("pinned", 0),
                                         ("pinned", 3)])
@pytest.mark.parametrize("n,i32", [(1000, True), (1001, False),
                                   (9000, True)])
def test_loads_from_any_device_pointer(where, shift, n, i32):
    g = synth.random_game(n, 2, 5, n)
    ref = orc.solve(g)
    keep = [_place(g["offsets"].astype(np.int32 if i32 else np.int64), where,
                   shift)] + \
        [_place(g[k], where, shift) for k in ("targets", "owner", "pri")]
    torch.cuda.synchronize()
    h = ctypes.c_void_p()
    s = torch.cuda.current_stream().cuda_stream
    assert lib().pg_load_csr(n, g["m"], *[p for _, p in keep],
                             PG_PTR_DEVICE | (PG_OFFSETS_I32 if i32 else 0),
                             s, ctypes.byref(h)) == PG_OK
    try:
        winner = torch.empty(n, dtype=torch.uint8, device="cuda")
        opts = SolveOpts(0, 0, PG_PTR_DEVICE | PG_KEEP_DUMMIES, 0, None, None,
                         0, 0, None, None, None, None)
        st = Stats()
        assert lib().pg_solve(h, ctypes.byref(opts), winner.data_ptr(), None,
                              None, ctypes.byref(st), s) == PG_OK
        np.testing.assert_array_equal(to_np(winner), ref["winner"])
        assert st.n_valuations == ref["n_valuations"]
    finally:
        lib().pg_free(h)


@pytest.mark.parametrize("where,shift", [("device", 0), ("device", 2),
                                         ("pinned", 0), ("pinned", 1)])
def test_polls_to_any_device_pointer(where, shift):
    games = [synth.random_game(n, 2, 5, n) for n in (50, 700, 3001)]
    with Batch(1 << 16, 1 << 18) as b:
        t = np.array(b.submit_many(games), np.int64)
        while b.step()[0] > 0:
            pass
        done = np.zeros(3, np.int32)
        out = [[_place(np.zeros(size * k, np.uint8), where, shift)
                for k, size in ((g["n"], 1), (2 * g["n"], 4), (2 * g["n"], 4))]
               for g in games]
        torch.cuda.synchronize()
        ptrs = [(ctypes.c_void_p * 3)(*[o[j][1] for o in out])
                for j in range(3)]
        st = (Stats * 3)()
        assert lib().pg_batch_poll_many(
            b._h, 3, t.ctypes.data, done.ctypes.data, *ptrs, st,
            PG_PTR_DEVICE) == PG_OK
    assert done.all()
    for g, o, s in zip(games, out, st):
        ref = orc.solve(g)
        na = s.n_aug
        for (buf, _), count, size, want in zip(
                o, (g["n"], na, na), (1, 4, 4),
                (ref["winner"], ref["sigma"], ref["tau_orig"])):
            raw = to_np(buf)[shift:shift + size * count].copy()
            got = raw if size == 1 else raw.view(np.int32)
            np.testing.assert_array_equal(got, want)

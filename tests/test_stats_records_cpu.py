"""A worker's statistics as a dict against the record's fields one by one."""
import ctypes
import random

import pytest

import paper_2601_18999_amd as K


@pytest.mark.parametrize("n", [0, 1, 7])
def test_records_hold_every_field(n):
    arr = (K.KvrWorkerStats * 7)()
    raw = random.Random(n).randbytes(ctypes.sizeof(arr))
    ctypes.memmove(arr, raw, len(raw))
    got = K._stats_dicts(arr, n)
    assert len(got) == n
    for s, d in zip(arr, got):
        want = {name: getattr(s, name) for name, _ in K.KvrWorkerStats._fields_}
        want["theta"] = list(s.theta)
        assert repr(d) == repr(want)  # keys in order, values and their types (a NaN too)

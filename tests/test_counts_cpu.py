"""Token counts as the binding hands them to the library: the whole list, whatever holds it."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

from paper_2609_33184_amd import specstream as ss

ROWS = [[5, 6], [7, 0], [2 ** 31 - 1, 1]]


class _Lib:
    """Stands for the library: keeps the counts found at the address passed."""

    def __init__(self, n):
        self.n = n

    def __getattr__(self, name):
        at = {"ss_attend_history_chunk": 3, "ss_attend_history_chunks": 4, "ss_pipeline_attend_chunk": 3,
              "ss_pipeline_attend_chunks": 4}[name]

        def call(*args):
            self.got = list((ctypes.c_int32 * self.n).from_address(args[at]))
            return ss.SS_OK
        return call


FORMS = [
    ("lists", lambda: ROWS),
    ("tuples", lambda: tuple(tuple(r) for r in ROWS)),
    ("floats", lambda: [[float(x) for x in r] for r in ROWS]),
    ("numpy", lambda: np.array(ROWS, dtype=np.int64)),
    ("numpy floats", lambda: np.array(ROWS, dtype=np.float64)),
    ("tensors", lambda: [torch.tensor(r) for r in ROWS]),
    ("iterators of ints", lambda: [iter(r) for r in ROWS]),
    ("iterators of floats", lambda: [iter([float(x) for x in r]) for r in ROWS]),
    ("a float behind ints", lambda: [iter(ROWS[0]), iter([7, 0.0]), iter(ROWS[2])]),
    ("texts", lambda: [[str(x) for x in r] for r in ROWS]),
]


@pytest.mark.parametrize("form", [f[1] for f in FORMS], ids=[f[0] for f in FORMS])
def test_counts_arrive_whole(form, monkeypatch):
    flat = [x for r in ROWS for x in r]
    lib = _Lib(len(flat))
    monkeypatch.setattr(ss, "load", lambda: lib)
    ss.ss_attend_history_chunks(1, [0] * 3, [0] * 3, form())
    assert lib.got == flat
    lib.got = None
    ss.ss_pipeline_attend_chunks(1, 1, 0, form())
    assert lib.got == flat
    for i, row in enumerate(ROWS):
        lib = _Lib(len(row))
        monkeypatch.setattr(ss, "load", lambda: lib)
        ss.ss_attend_history_chunk(1, 0, 0, form()[i])
        assert lib.got == row
        lib.got = None
        ss.ss_pipeline_attend_chunk(1, 1, 0, form()[i])
        assert lib.got == row


@pytest.mark.parametrize("count", [2 ** 31, 2 ** 32 + 5, -2 ** 31 - 1, float(2 ** 32 + 5)])
def test_counts_beyond_32_bits_are_refused(count, monkeypatch):
    monkeypatch.setattr(ss, "load", lambda: pytest.fail("the library was called"))
    monkeypatch.setattr(ss, "ss_status_string", lambda s: "refused")
    for call in (lambda: ss.ss_attend_history_chunk(1, 0, 0, [1, count]),
                 lambda: ss.ss_attend_history_chunks(1, [], [], [[1, count]]),
                 lambda: ss.ss_pipeline_attend_chunk(1, 1, 0, [1, count]),
                 lambda: ss.ss_pipeline_attend_chunks(1, 1, 0, [[1, count]])):
        with pytest.raises(ss.SpecStreamError) as e:
            call()
        assert e.value.status == ss.SS_ERR_INVALID_ARGUMENT

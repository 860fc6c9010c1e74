"""The streams of a captured step come round robin from a pool: none may be
one that the step already uses."""
import itertools

import pytest
import torch

from paper_2303_12980_amd import gmp


class _Fake:
    def __init__(self, h):
        self.cuda_stream = h


@pytest.mark.parametrize("start", range(3))
def test_distinct_streams(monkeypatch, start):
    pool = itertools.cycle([1, 2, 3])
    for _ in range(start):
        next(pool)
    monkeypatch.setattr(torch.cuda, "Stream", lambda: _Fake(next(pool)))
    cur = _Fake(1)
    side = gmp._stream_beside(cur)
    rev = gmp._stream_beside(cur, side)
    assert len({cur.cuda_stream, side.cuda_stream, rev.cuda_stream}) == 3


def test_exhausted_pool_raises(monkeypatch):
    monkeypatch.setattr(torch.cuda, "Stream", lambda: _Fake(1))
    with pytest.raises(RuntimeError):
        gmp._stream_beside(_Fake(1))

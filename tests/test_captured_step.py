"""A captured step's streams, with torch's CUDA calls replaced (CPU): the capture
runs on a stream that is not the caller's, and a second stream inside the
capture is refused, by the autotuner too, whatever an older cache holds."""
import contextlib
import itertools
import json
import types

import pytest
import torch

from paper_2303_12980_amd import _lib, autotune, gmp


class _Stream:
    def __init__(self, h):
        self.cuda_stream = h

    def wait_stream(self, other):
        pass


def _pieces(reverse=True):
    plan = types.SimpleNamespace(n_features=2, n_components=3, dtype=torch.float32,
                                 batch_workspace_bytes=lambda b, c: 8, set_tuning=lambda **k: None)
    species = torch.zeros(4, dtype=torch.int32)
    batch = types.SimpleNamespace(species=species, n_centres=4, n_total=4, n_structs=1, n_points=0, xyz=None,
                                  cell=None, atom_offsets=None, pbc=None, occupancy=None, point_offsets=None,
                                  pxyz=None)
    ws = types.SimpleNamespace(buf=None, get=lambda n: None)
    nb = types.SimpleNamespace(capacity=1, n_pairs=1, reverse=species if reverse else None, offsets=None, j=None,
                               shift=None, bucket_start=None, sigma_end=None, wrap=None, rw=None, order=None,
                               slot=None)
    return plan, batch, ws, nb


@pytest.fixture
def cuda(monkeypatch):
    """torch.cuda with streams of a pool of three, the caller on the first."""
    rec = types.SimpleNamespace(current=_Stream(1), captured=[], ran=[])
    pool = itertools.cycle([1, 2, 3])

    @contextlib.contextmanager
    def on(s):
        before, rec.current = rec.current, s
        yield
        rec.current = before

    @contextlib.contextmanager
    def graph(g, stream=None):
        rec.captured.append(stream)
        with on(stream):
            yield

    monkeypatch.setattr(torch.cuda, "Stream", lambda: _Stream(next(pool)))
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: rec.current)
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch.cuda, "graph", graph)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    monkeypatch.setattr(torch.cuda, "CUDAGraph", lambda: object())
    monkeypatch.setattr(gmp.CapturedStep, "_run", lambda self: rec.ran.append(rec.current.cuda_stream))
    return rec


@pytest.mark.parametrize("backward", [False, True])
def test_capture_runs_beside_the_callers_stream(cuda, backward):
    gmp.CapturedStep(*_pieces(), backward=backward)
    assert [s.cuda_stream for s in cuda.captured] == [2]
    assert cuda.ran == [2, 2]  # the warm-up and the capture
    assert cuda.current.cuda_stream == 1


def test_second_stream_inside_the_capture_is_refused(cuda):
    with pytest.raises(_lib.GMPError) as e:
        gmp.CapturedStep(*_pieces(), backward=True, concurrent_reverse=True)
    assert e.value.status == _lib.GMP_E_UNSUPPORTED
    assert not cuda.ran and not cuda.captured
    # without an effect it is taken, as before
    gmp.CapturedStep(*_pieces(), backward=False, concurrent_reverse=True)
    gmp.CapturedStep(*_pieces(reverse=False), backward=True, concurrent_reverse=True)
    assert len(cuda.captured) == 2


def test_autotuner_keeps_one_stream(monkeypatch, tmp_path):
    plan, batch, ws, nb = _pieces()
    monkeypatch.setattr(gmp, "build_neighbors", lambda *a, **k: nb)
    monkeypatch.setattr(autotune, "tuning_key", lambda *a: "key")
    path = tmp_path / "tune.json"
    path.write_text(json.dumps({"key": dict(tuning=dict(chunk_pairs=512), ms=1.0, concurrent_reverse=True)}))
    r = autotune.autotune(plan, batch, ws, cache_path=str(path))
    assert r["cached"] and r["concurrent_reverse"] is False
    with pytest.raises(_lib.GMPError):
        autotune.autotune(plan, batch, ws, cache_path=str(path), streams=True)
    # a search captures nothing
    monkeypatch.setattr(autotune, "_time_config", lambda *a: 1.0)
    monkeypatch.setattr(gmp, "CapturedStep", None)
    r = autotune.autotune(plan, batch, ws, cache_path=str(tmp_path / "none.json"))
    assert not r["cached"] and r["concurrent_reverse"] is False

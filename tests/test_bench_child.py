"""The benchmark's part that runs in a process of its own: a child that fails is
named in the line and gives the benchmark its exit status."""
import subprocess
import types

import pytest

import bench


@pytest.mark.parametrize("rc,out,status", [(0, 'note\n{"C4": 1}\n', 0), (1, "", 1), (-11, "", 1), (139, "", 139),
                                           (0, "", 1)])
def test_status_of_the_child(monkeypatch, rc, out, status):
    monkeypatch.setattr(subprocess, "run", lambda *a, **k: types.SimpleNamespace(returncode=rc, stdout=out))
    line, got = bench.other_workloads_apart()
    assert got == status
    assert line == ({"C4": 1} if status == 0 else {"error": f"exit status {rc}"})

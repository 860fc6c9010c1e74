import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU")
    config.addinivalue_line("markers", "slow: longer CPU test")


# Tests of a captured step whose reverse search runs on a second stream: the
# mode is switched off (CapturedStep refuses it), because the replay of such
# steps has ended the host process and the cause is not known.
TWO_STREAM_STEPS = (
    "test_gpu_graph.py::test_graph_replay_matches_eager[fp32c-True]",
    "test_gpu_graph.py::test_graph_replay_growing_pair_count[False-True]",
    "test_gpu_graph.py::test_autotune_choice_and_cache",
)


def pytest_collection_modifyitems(items):
    skip = pytest.mark.skip(reason="captured steps on two streams are switched off: a host fault of unknown cause")
    for item in items:
        if item.nodeid.endswith(TWO_STREAM_STEPS):
            item.add_marker(skip)

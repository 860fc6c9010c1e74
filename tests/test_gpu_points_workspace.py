"""The workspace of reference points: the counters of the neighbour build belong to
the centres, so a few points in many atoms do not pay for 32 ranges per atom."""
import numpy as np
import pytest

import gmp_synth as gs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_bytes_per_atom():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_12980_amd as g
    g.load()
    probes = gs.small_probes(np.random.default_rng(0), orders=(0,), n_sigmas=1, n_elements=1)
    plan = g.GMPPlan.from_probes(probes, "fp32c")
    few, many = (plan.workspace_bytes(1, n, 4096, n_points=64) for n in (1_000_000, 2_000_000))
    # positions, bins, order, packed copies and per-centre arrays: about 256 bytes an
    # atom; one counter per atom and range would add 128
    assert (many - few) / 1e6 < 280

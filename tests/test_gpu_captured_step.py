"""Captured steps made and replayed on a caller's own stream, and the autotuner's
search and cache, on the GPU."""
import json

import numpy as np
import pytest

import gmp_synth as gs
import oracle
from gpu_helpers import assert_features

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def g():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_12980_amd as g
    g.load()
    return g


@pytest.mark.parametrize("steps", [1, 40])
def test_step_on_a_callers_stream(g, steps):
    """Every replay equals the eager result bit for bit, also of a step captured
    after torch's pool of streams has gone round."""
    rng = np.random.default_rng(41)
    struct = gs.small_periodic(rng, n_atoms=30, n_elements=2, density=0.05, dmin=1.2)
    probes = gs.small_probes(rng, n_sigmas=3, n_elements=2)
    b = gs.make_batch([struct])
    plan = g.GMPPlan.from_probes(probes, "fp32c")
    db = g.DeviceBatch.from_batch(b)
    ws = g.Workspace()
    nb = g.build_neighbors(plan, db, ws)
    G = torch.as_tensor(rng.standard_normal((30, probes.n_features)), device="cuda").to(plan.dtype)
    F0, mu0 = g.features(plan, db, nb, ws)
    gp0, gc0 = g.features_backward(plan, db, nb, ws, mu0, F0, G)
    torch.cuda.synchronize()
    mine = torch.cuda.Stream()
    with torch.cuda.stream(mine):
        for _ in range(steps):
            step = g.CapturedStep(plan, db, ws, g.build_neighbors(plan, db, ws), backward=True, G=G)
        for _ in range(3):
            for t in (step.F, step.mu, step.gpos, step.gcell):
                t.zero_()
            step.replay()
            mine.synchronize()
            for got, ref in ((step.F, F0), (step.mu, mu0), (step.gpos, gp0.t().reshape(-1)),
                             (step.gcell, gc0.reshape(-1))):
                assert torch.equal(got, ref)
        step.check_status(mine)


def test_autotuner_search_and_cache(g, tmp_path):
    from paper_2303_12980_amd import autotune
    b, probes = gs.config("C1")
    plan = g.GMPPlan.from_probes(probes, "fp32c")
    db = g.DeviceBatch.from_batch(b)
    ws = g.Workspace()
    cache = str(tmp_path / "tune.json")
    cands = [dict(chunk_pairs=0, bin_divisor=2, blocks_per_cu=0, adj_items=0, sigma_groups=1),
             dict(chunk_pairs=256, bin_divisor=3, blocks_per_cu=0, adj_items=2, sigma_groups=2)]
    r = autotune.autotune(plan, db, ws, candidates=cands, reps=2, cache_path=cache)
    assert not r["cached"] and r["concurrent_reverse"] is False
    assert r["tuning"] == r["tried"][autotune.choose(r["tried"])]["tuning"] == plan.get_tuning()
    with open(cache) as f:
        assert r["key"] in json.load(f)
    plan2 = g.GMPPlan.from_probes(probes, "fp32c")
    r2 = autotune.autotune(plan2, db, ws, candidates=cands, cache_path=cache)
    assert r2["cached"] and plan2.get_tuning() == r["tuning"] and r2["concurrent_reverse"] is False
    nb = g.build_neighbors(plan2, db, ws)
    F, _ = g.features(plan2, db, nb, ws)
    assert_features(F.cpu().numpy(), oracle.features_batch(b, probes), probes.tau, 1e-5)

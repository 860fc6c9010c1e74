"""Primitives so wide that they are flat over the structure (beta = 1e-30): a
lane of the overlap kernel that has no pair of a slot must add nothing, whatever
the slot's exponents.  Isolated structures whose lists end inside a wavefront's
step, against the FP64 oracle (tolerances of the parity tests)."""
import numpy as np
import pytest

import gmp_synth as gs
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = {"fp64": 1e-11, "fp32c": 1e-5, "fp32w": 1e-5}


@pytest.mark.parametrize("prec", ["fp64", "fp32w", "fp32c"])
@pytest.mark.parametrize("lmax", [1, 3, 4])
@pytest.mark.parametrize("n", [5, 65, 100])
def test_flat_primitives(prec, lmax, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_12980_amd as g
    g.load()
    rng = np.random.default_rng(n)
    struct = gs.small_cluster(rng, n_atoms=n, n_elements=2, radius=1.1 * n ** (1.0 / 3.0) + 1.0, dmin=1.0)
    probes = gs.Probes(np.arange(-1, lmax + 1, dtype=np.int32), np.geomspace(0.4, 1.2, 5), np.array([0, 2, 4], np.int32),
                       np.array([1.0, 1e-2, 0.7, 2e-2]), np.array([0.3, 1e-30, 0.5, 1e-30]), 1e-11)
    plan = g.GMPPlan.from_probes(probes, prec)
    db = g.DeviceBatch.from_batch(gs.make_batch([struct]))
    ws = g.Workspace()
    nb = g.build_neighbors(plan, db, ws)
    assert nb.n_pairs == n * n
    Fr, mur = oracle.features(struct, probes, with_mu=True)
    F, mu = g.features(plan, db, nb, ws)
    F0, _ = g.features(plan, db, nb, ws, with_components=False)
    for got, ref in ((F, Fr), (F0, Fr), (mu, mur)):
        scale = np.maximum(np.abs(ref).max(0), probes.tau)
        assert (np.abs(got.double().cpu().numpy() - ref) / scale).max() <= TOL[prec]

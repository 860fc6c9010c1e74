"""The overlap and adjoint kernels at the edges of their work split: cutoff
slots that do not fill the last pass (every slot count from 1 up, with and
without the density slot), every highest order, lists that end one pair before,
at and after a wavefront's or two wavefronts' worth of pairs, and every stride of
the primitive tables, against the FP64 oracle.

Tolerances as in the parity tests, relative to the largest value of each
feature column or gradient: 1e-11 (FP64), 1e-5 (FP32 modes)."""
import numpy as np
import pytest

import gmp_synth as gs
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TOL = {"fp64": 1e-11, "fp32c": 1e-5, "fp32w": 1e-5}


@pytest.fixture(scope="module")
def g():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_12980_amd as g
    g.load()
    return g


def _check(g, struct, probes, prec, occupancy=None, **tuning):
    b = gs.make_batch([struct], None if occupancy is None else [occupancy])
    plan = g.GMPPlan.from_probes(probes, prec)
    if tuning:
        plan.set_tuning(**tuning)
    ws = g.Workspace()
    db = g.DeviceBatch.from_batch(b)
    nb = g.build_neighbors(plan, db, ws)
    F, mu = g.features(plan, db, nb, ws)
    Fr, mur = oracle.features(struct, probes, with_mu=True, occupancy=occupancy)
    G = gs.upstream_gradient(5, *Fr.shape)
    if prec != "fp64":
        G = G.astype(np.float32).astype(np.float64)
    gp, gc = g.features_backward(plan, db, nb, ws, mu, F, torch.as_tensor(G, device="cuda"))
    torch.cuda.synchronize()
    rp, rc, _ = oracle.grad(struct, probes, G, occupancy=occupancy)
    for got, ref in ((F, Fr), (mu, mur)):
        scale = np.maximum(np.abs(ref).max(0), probes.tau)
        assert (np.abs(got.double().cpu().numpy() - ref) / scale).max() <= TOL[prec]
    scale = max(np.abs(rp).max(), np.abs(rc).max(), probes.tau)
    assert np.abs(gp.cpu().numpy() - rp).max() <= TOL[prec] * scale
    assert np.abs(gc.cpu().numpy()[0] - rc).max() <= TOL[prec] * scale
    return nb


@pytest.mark.parametrize("prec", ["fp32c", "fp64"])
@pytest.mark.parametrize("lmax", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("density", [False, True])
def test_every_slot_count(g, prec, lmax, density):
    rng = np.random.default_rng(900 + 10 * lmax + density)
    struct = gs.small_periodic(rng, n_atoms=9, n_elements=2, density=0.06)
    for n_sig in range(1, 10):
        orders = ([-1] if density else []) + list(range(lmax + 1))
        probes = gs.small_probes(rng, orders=orders, n_sigmas=n_sig, n_elements=2)
        _check(g, struct, probes, prec)


@pytest.mark.parametrize("prec", ["fp32c", "fp32w", "fp64"])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 127, 128, 129, 193])
def test_list_ends(g, prec, n):
    """Clusters whose lists hold all n atoms for every slot."""
    rng = np.random.default_rng(n)
    struct = gs.small_cluster(rng, n_atoms=n, n_elements=3, radius=1.1 * n ** (1.0 / 3.0) + 1.0, dmin=1.0)
    probes = gs.small_probes(rng, n_sigmas=5, n_elements=3, tau=1e-14, sig_range=(0.8, 1.5), beta_range=(0.02, 0.06))
    nb = _check(g, struct, probes, prec, occupancy=rng.uniform(0.3, 1.0, n))
    assert nb.n_pairs == n * n
    _check(g, struct, probes, prec, chunk_pairs=64, sigma_groups=2)


@pytest.mark.parametrize("prec", ["fp32c", "fp64"])
@pytest.mark.parametrize("prims", [1, 4, 5, 8, 9, 16])
def test_primitive_counts(g, prec, prims):
    rng = np.random.default_rng(prims)
    struct = gs.small_periodic(rng, n_atoms=7, n_elements=2, density=0.05)
    _check(g, struct, gs.small_probes(rng, n_sigmas=3, n_elements=2, n_prims=prims), prec)
    _check(g, struct, gs.small_probes(rng, n_sigmas=3, n_elements=2, n_prims=(1, prims)), prec,
           occupancy=rng.uniform(0.3, 1.0, 7))

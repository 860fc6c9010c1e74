"""The neighbour build where its route changes: the one-workgroup cell list
against the general one (around 1024 atoms, points or structures), the number of
index ranges a bucket is split into (by cutoff slots x species), and ranges on
both sides of the length up to which they are ordered by counting.  Lists,
bucket starts, prefix ends and the reverse index are integers and must equal the
oracle's."""
import numpy as np
import pytest

import gmp_synth as gs
import oracle
from gpu_helpers import check_lists_many, check_reverse

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def g():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_12980_amd as g
    g.load()
    return g


def _build(g, structs, probes):
    b = gs.make_batch(structs)
    plan = g.GMPPlan.from_probes(probes, "fp32c")
    ws = g.Workspace()
    db = g.DeviceBatch.from_batch(b)
    nb = g.build_neighbors(plan, db, ws)
    check_reverse(nb)
    F0, _ = g.features(plan, db, nb, ws, with_components=False)
    F1, _ = g.features(plan, db, nb, ws)
    scale = F1.abs().amax(0).clamp_min(probes.tau)
    assert float(((F0 - F1).abs() / scale).max()) <= 1e-5
    # a no-sync rebuild of the same batch gives the same lists
    ref = [t.clone() for t in (nb.offsets, nb.j[:nb.n_pairs], nb.shift[:nb.n_pairs], nb.reverse[:nb.n_pairs])]
    n = nb.n_pairs
    g.rebuild_neighbors_nosync(plan, db, ws, nb)
    g.check_status(ws)
    for a, c in zip(ref, (nb.offsets, nb.j[:n], nb.shift[:n], nb.reverse[:n])):
        assert torch.equal(a, c)
    return b, nb


@pytest.mark.parametrize("n", [1, 2, 1023, 1024, 1025])
def test_one_structure(g, n):
    rng = np.random.default_rng(n)
    struct = gs.small_periodic(rng, n_atoms=n, n_elements=2, density=0.05, dmin=1.2)
    probes = gs.small_probes(rng, n_sigmas=3, n_elements=2)
    b, nb = _build(g, [struct], probes)
    check_lists_many(nb, b, probes, 0, np.arange(0, n, max(1, n // 64)))


@pytest.mark.parametrize("n_structs", [3, 1024, 1025])
def test_many_structures(g, n_structs):
    """One or two atoms each (and the last one empty): few atoms, many structures."""
    rng = np.random.default_rng(n_structs)
    cell = np.eye(3) * 5.0
    structs = []
    for s in range(n_structs):
        k = 0 if s == n_structs - 1 else (1 if n_structs > 3 else 2)
        structs.append((rng.random((k, 3)) * 5.0, np.zeros(k, np.int32), cell, 7 if s % 2 else 0))
    probes = gs.small_probes(rng, orders=(0, 1), n_sigmas=2, n_elements=1)
    b, nb = _build(g, structs, probes)
    for s in range(0, n_structs - 1, max(1, n_structs // 16)):
        check_lists_many(nb, b, probes, s)


@pytest.mark.parametrize("slots,species", [(1, 1), (6, 8), (7, 7), (16, 6), (9, 11), (16, 12), (15, 13)])
def test_range_counts(g, slots, species):
    rng = np.random.default_rng(100 * slots + species)
    struct = gs.small_periodic(rng, n_atoms=90, n_elements=species, density=0.06, dmin=1.2)
    probes = gs.small_probes(rng, orders=(0, 1), n_sigmas=slots, n_elements=species)
    b, nb = _build(g, [struct], probes)
    check_lists_many(nb, b, probes, 0)


@pytest.mark.parametrize("n", [128, 129, 1000, 1030, 1100])
def test_counted_and_sorted_ranges(g, n):
    """Isolated structures of one species and one slot: every list is one bucket
    of n entries, its ranges n/8 long (up to 128 entries ordered by counting)."""
    rng = np.random.default_rng(n)
    pos = rng.random((n, 3)) * 2.0
    struct = (pos, np.zeros(n, np.int32), np.zeros((3, 3)), 0)
    probes = gs.small_probes(rng, orders=(0,), n_sigmas=1, n_elements=1, tau=1e-14, beta_range=(0.02, 0.06))
    b, nb = _build(g, [struct], probes)
    assert nb.n_pairs == n * n
    check_lists_many(nb, b, probes, 0, np.arange(0, n, 17))


@pytest.mark.parametrize("n", [8, 1500])
def test_faults_are_reported(g, n):
    """A singular lattice, also of a structure without atoms, and a non-finite coordinate."""
    rng = np.random.default_rng(n)
    probes = gs.small_probes(rng, orders=(0,), n_sigmas=1, n_elements=1)
    plan = g.GMPPlan.from_probes(probes, "fp32c")
    ok = (rng.random((n, 3)) * 30.0, np.zeros(n, np.int32), np.eye(3) * 30.0, 7)
    flat = np.diag([30.0, 30.0, 0.0])
    for bad in ((ok[0], ok[1], flat, 7), (np.zeros((0, 3)), np.zeros(0, np.int32), flat, 7),
                (np.where(np.arange(3 * n).reshape(n, 3) == 4, np.nan, ok[0]), ok[1], ok[2], 7)):
        with pytest.raises(g.GMPError):
            g.build_neighbors(plan, g.DeviceBatch.from_batch(gs.make_batch([ok, bad])), g.Workspace())
    g.build_neighbors(plan, g.DeviceBatch.from_batch(gs.make_batch([ok])), g.Workspace())

"""The number of index ranges a bucket is split into follows the plan's buckets,
the atoms per structure and the capacity: lists, bucket starts, prefix ends and
the reverse index are the oracle's at the edges of each, for atoms in random and in
spatial order, and the same at every capacity."""
import numpy as np
import pytest

import gmp_synth as gs
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


def _check(g, structs, probes, **kw):
    b = gs.make_batch(structs)
    plan = g.GMPPlan.from_probes(probes, "fp32c")
    ws = g.Workspace()
    db = g.DeviceBatch.from_batch(b)
    nb = g.build_neighbors(plan, db, ws, **kw)
    check_reverse(nb)
    return b, db, plan, nb


@pytest.mark.parametrize("slots,species", [(1, 1), (3, 4), (1, 13), (4, 6), (5, 5), (6, 8)])
@pytest.mark.parametrize("n", [31, 32, 70])
def test_most_ranges(g, slots, species, n):
    """32 ranges up to 12 buckets, 16 up to 24, 8 up to 48; structures around 32 atoms."""
    rng = np.random.default_rng(1000 * slots + 10 * species + n)
    probes = gs.small_probes(rng, orders=(0, 1), n_sigmas=slots, n_elements=species, tau=1e-13, beta_range=(0.1, 0.4))
    struct = gs.small_periodic(rng, n_atoms=n, n_elements=species, density=0.06, dmin=1.2)
    b, _, _, nb = _check(g, [struct], probes)
    assert nb.n_pairs > 384 * n  # long lists: the atoms and the buckets decide
    check_lists_many(nb, b, probes, 0, np.arange(0, n, 3))


def test_every_capacity_gives_the_same_lists(g):
    """Room for a multiple of the lists (some 20 entries, 6 buckets) decides the
    ranges: from two or four at the exact count to 32."""
    rng = np.random.default_rng(5)
    probes = gs.small_probes(rng, orders=(0, 1), n_sigmas=3, n_elements=2, tau=1e-3, beta_range=(1.0, 3.0))
    structs = [gs.small_periodic(rng, n_atoms=n, n_elements=2, density=0.06, dmin=1.2) for n in (33, 64, 200)]
    b, db, plan, nb = _check(g, structs, probes)
    for s in range(3):
        check_lists_many(nb, b, probes, s)
    n = nb.n_pairs
    for f in (1, 2, 4, 8, 32):
        for late in (False, True):
            ws = g.Workspace()
            nb2 = g.build_neighbors(plan, db, ws, capacity=f * n, defer_reverse=late)
            if late:
                g.build_reverse(plan, db, ws, nb2)
            g.check_status(ws)
            for a, c in ((nb.offsets, nb2.offsets), (nb.j[:n], nb2.j[:n]), (nb.shift[:n], nb2.shift[:n]),
                         (nb.reverse[:n], nb2.reverse[:n]), (nb.bucket_start, nb2.bucket_start),
                         (nb.sigma_end, nb2.sigma_end)):
                assert torch.equal(a, c)


@pytest.mark.parametrize("slots,species", [(2, 2), (6, 4), (8, 6)])
def test_atoms_in_spatial_order(g, slots, species):
    """3000 atoms listed layer by layer: a centre's neighbours share few ranges, some
    longer than the counting takes."""
    rng = np.random.default_rng(slots)
    pos, spec, cell, pbc = gs.small_periodic(rng, n_atoms=3000, n_elements=species, density=0.06, dmin=1.2)
    f = np.floor((pos @ np.linalg.inv(cell) % 1.0) * 12).astype(int)
    order = np.lexsort((f[:, 2], f[:, 1], f[:, 0]))
    probes = gs.small_probes(rng, orders=(0, 1), n_sigmas=slots, n_elements=species, tau=1e-11, beta_range=(0.2, 0.6))
    b, _, _, nb = _check(g, [(pos[order], spec[order], cell, pbc)], probes)
    check_lists_many(nb, b, probes, 0, np.arange(0, 3000, 47))

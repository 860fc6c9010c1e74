"""Positions that diverged after the lists were built: a non-finite atom spoils the
features of the centres and cutoff slots whose lists hold it, and no others (several
slots share a walk over a list, one of them may end before the atom)."""
import numpy as np
import pytest

import gmp_synth as gs
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["fp32c", "fp32w", "fp64"])
@pytest.mark.parametrize("lmax", [1, 2, 3, 4])
@pytest.mark.parametrize("value", [float("nan"), 1e40])
def test_spoilt_slots(prec, lmax, value):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_12980_amd as g
    g.load()
    rng = np.random.default_rng(lmax)
    n, bad = 60, 17
    struct = gs.small_cluster(rng, n_atoms=n, n_elements=2, radius=7.0, dmin=1.2)
    # slots of clearly different cutoffs, about 3 to 9 A
    probes = gs.Probes(np.arange(lmax + 1, dtype=np.int32), np.array([0.3, 0.6, 1.0, 1.4, 1.8]), np.array([0, 1, 2], np.int32),
                       np.array([1.0, 0.8]), np.array([2.0, 2.5]), 1e-5)
    rc2 = oracle.cutoffs(probes)
    assert np.all(np.diff(rc2) > 1.0)
    plan = g.GMPPlan.from_probes(probes, prec)
    db = g.DeviceBatch.from_batch(gs.make_batch([struct]))
    ws = g.Workspace()
    nb = g.build_neighbors(plan, db, ws)
    d2 = ((struct[0] - struct[0][bad]) ** 2).sum(1)
    F0, _ = g.features(plan, db, nb, ws)
    xyz = db.xyz.clone()
    xyz[0, bad] = value
    for comps in (True, False):
        F, _ = g.features(plan, db, nb, ws, with_components=comps, xyz=xyz)
        F = F.double().cpu().numpy()
        for l in range(lmax + 1):
            for s in range(5):
                col = l * 5 + s
                holds = d2 <= rc2[s]  # the centre's list holds the atom within the slot (itself included)
                if np.isnan(value):
                    assert np.isnan(F[holds, col]).all()
                assert np.isfinite(F[~holds, col]).all(), (l, s)
                ref = F0[:, col].double().cpu().numpy()
                assert np.abs(F[~holds, col] - ref[~holds]).max(initial=0.0) <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("prec", ["fp32c", "fp32w", "fp64"])
@pytest.mark.parametrize("what", ["occupancy", "cell"])
def test_spoilt_by_occupancies_and_lattice(prec, what):
    """The same for an occupancy that is no number, and for a lattice that has grown
    beyond any cutoff: slots of pairs within the cell alone keep their features."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_12980_amd as g
    g.load()
    rng = np.random.default_rng(3)
    n, bad, lmax, S = 120, 31, 3, 5
    struct = gs.small_periodic(rng, n_atoms=n, n_elements=2, density=0.05, dmin=1.2)
    cell = struct[2]
    struct = ((struct[0] @ np.linalg.inv(cell) % 1.0) @ cell, struct[1], cell, struct[3])  # no lattice wrap
    probes = gs.Probes(np.arange(lmax + 1, dtype=np.int32), np.array([0.3, 0.6, 1.0, 1.4, 1.8]), np.array([0, 1, 2], np.int32),
                       np.array([1.0, 0.8]), np.array([2.0, 2.5]), 1e-5)
    occ = rng.uniform(0.5, 1.0, n)
    plan = g.GMPPlan.from_probes(probes, prec)
    db = g.DeviceBatch.from_batch(gs.make_batch([struct], [occ]))
    ws = g.Workspace()
    nb = g.build_neighbors(plan, db, ws)
    F0, _ = g.features(plan, db, nb, ws)
    F0 = F0.double().cpu().numpy()
    # per centre and slot: does the prefix hold the bad atom / a pair outside the cell?
    offs, slot = nb.offsets.cpu().numpy(), nb.slot.cpu().numpy()
    end = nb.sigma_end.view(-1, S).cpu().numpy()
    J, w = nb.j.cpu().numpy(), nb.shift.cpu().numpy()
    spoilt = np.zeros((n, S), bool)
    for i in range(n):
        o = offs[slot[i]]
        for s in range(S):
            e = o + end[slot[i], s]
            spoilt[i, s] = (J[o:e] == bad).any() if what == "occupancy" else ((w[o:e] & 0xffffff) != 0).any()
    assert spoilt.any() and not spoilt.all()
    kw = {}
    if what == "occupancy":
        db.occupancy[bad] = float("nan")
    else:
        kw["cell"] = db.cell * 1e25
    for comps in (True, False):
        F, _ = g.features(plan, db, nb, ws, with_components=comps, **kw)
        F = F.double().cpu().numpy().reshape(n, lmax + 1, S)
        ref = F0.reshape(n, lmax + 1, S)
        for s in range(S):
            ok = ~spoilt[:, s]
            if what == "occupancy":
                assert np.isnan(F[~ok, :, s]).all()
            assert np.isfinite(F[ok, :, s]).all(), s
            assert np.abs(F[ok, :, s] - ref[ok, :, s]).max(initial=0.0) <= 1e-5 * np.abs(ref[:, :, s]).max()

"""Atom indices past 2^27: reference points in the last structure of a batch of
2^27 + 40 atoms give the lists and the features that they give in that structure
alone, the neighbour indices shifted by the atoms before it."""
import numpy as np
import pytest

import gmp_synth as gs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_points_past_two_to_the_27_atoms():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_12980_amd as g
    g.load()
    if torch.cuda.mem_get_info()[0] < 200 << 30:
        pytest.skip("needs 200 GB of free GPU memory")
    rng = np.random.default_rng(27)
    struct = gs.small_periodic(rng, n_atoms=40, n_elements=2, density=0.05, dmin=1.2)
    probes = gs.small_probes(rng, orders=(0, 1), n_sigmas=1, n_elements=2)
    pts = rng.random((50, 3)) @ struct[2]
    small = g.DeviceBatch.from_batch(gs.make_batch([struct])).with_points(pts, [0, 50])
    per, before = 32, 1 << 27  # isolated structures of 32 atoms in front
    n_s = before // per
    big = g.DeviceBatch.__new__(g.DeviceBatch)
    big.__dict__.update(small.__dict__)
    dev = small.species.device
    big.atom_offsets = torch.cat([torch.arange(n_s + 1, dtype=torch.int64, device=dev) * per,
                                  torch.tensor([before + 40], device=dev)])
    big.point_offsets = torch.zeros(n_s + 2, dtype=torch.int64, device=dev)
    big.point_offsets[-1] = 50
    big.xyz = torch.zeros((3, before + 40), dtype=torch.float64, device=dev)
    big.xyz[:, before:] = small.xyz
    big.species = torch.zeros(before + 40, dtype=torch.int32, device=dev)
    big.species[before:] = small.species
    big.cell = torch.zeros((n_s + 1, 9), dtype=torch.float64, device=dev)
    big.cell[-1] = small.cell[0]
    big.pbc = torch.zeros(n_s + 1, dtype=torch.uint8, device=dev)
    big.pbc[-1] = small.pbc[0]
    big.n_structs, big.n_atoms = n_s + 1, before + 40
    plan = g.GMPPlan.from_probes(probes, "fp32c")
    ws = g.Workspace()
    ref = g.build_neighbors(plan, small, ws)
    Fref, _ = g.features(plan, small, ref, ws)
    torch.cuda.synchronize()
    wb = g.Workspace()
    nb = g.build_neighbors(plan, big, wb, capacity=ref.n_pairs + 64)
    F, _ = g.features(plan, big, nb, wb)
    torch.cuda.synchronize()
    n = ref.n_pairs
    assert nb.n_pairs == n > 0
    assert torch.equal(nb.offsets, ref.offsets)
    assert torch.equal(nb.j[:n].long(), ref.j[:n].long() + before)
    assert torch.equal(nb.shift[:n], ref.shift[:n])
    assert torch.equal(F, Fref)
    del nb, wb, big
    torch.cuda.empty_cache()

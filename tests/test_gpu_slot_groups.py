"""Groups of cutoff slots share a chunk's row of partial moments: they need no
more scratch than one group, and give the same bits."""
import ctypes

import pytest

import gmp_synth as gs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", ["fp32c", "fp64"])
def test_slot_groups_take_no_scratch(prec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2303_12980_amd as g
    L = g.load()
    b, p = gs.config("C2")  # its rows fill a quarter of the fixed array
    plan = g.GMPPlan.from_probes(p, prec)
    db = g.DeviceBatch.from_batch(b)
    ws = g.Workspace()
    nb = g.build_neighbors(plan, db, ws, reverse=False)
    F1, mu1 = g.features(plan, db, nb, ws)
    size = plan.batch_workspace_bytes(db, nb.capacity)
    for groups in (2, 16):
        plan.set_tuning(sigma_groups=groups)
        assert plan.batch_workspace_bytes(db, nb.capacity) == size
        F, mu = torch.full_like(F1, float("nan")), torch.full_like(mu1, float("nan"))
        bd, nd = db.desc(), nb.desc()
        st = L.gmp_features_noalloc(plan.handle, ctypes.byref(bd), ctypes.byref(nd), ctypes.c_void_p(F.data_ptr()),
                                    ctypes.c_void_p(mu.data_ptr()),
                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert st == 0, L.gmp_last_error()
        torch.cuda.synchronize()
        assert torch.equal(F, F1) and torch.equal(mu, mu1)

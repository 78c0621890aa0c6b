"""btl_forward_noalloc at the limit of its staging (1 MiB a slot): batches of
many small fields.  A field takes 336 B of the field table, 48 B of the phase
table's index and 8 B per workgroup, with two-step passes 376 B more; what does
not fit with passes runs in single steps.  M_final bit for bit against
btl_forward, E to 1e-13 (FP64 sums of terms <= 1 in another order)."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_q,passes", [(1300, (2, 1)), (1400, (0, 5)), (2600, (0, 5))])
def test_staging_limit(n_q, passes):
    import torch
    import paper_1907_00908_amd as btl
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    btl.load_library()
    cfg = w.make_config("cfg1", n=(2, 2, 2), K=5)
    cfg["gG0"] = np.array([0.7, -0.4, 0.59]) * np.linspace(0.01, 0.05, n_q)[:, None]
    cfg["q_geom"] = np.zeros(n_q, np.int32)
    print(f"GPU staging limit {n_q}", flush=True)
    out = []
    for noalloc in (True, False):
        sim = btl.Simulator(cfg["geoms"], cfg["bc"], "f32")
        try:
            E, M = sim.forward(cfg["dt"], cfg["D"], cfg["T2"], cfg["kappa"], cfg["f"], cfg["gG0"],
                               cfg["q_geom"], want_M=True, noalloc=noalloc)
            if noalloc:
                assert btl.btl_get_forward_passes(sim._h) == passes
            torch.cuda.synchronize()
            out.append((E.cpu().numpy(), torch.cat([m.reshape(-1) for m in M]).cpu().numpy()))
        finally:
            sim.close()
    assert np.array_equal(out[0][1], out[1][1])
    assert np.max(np.abs(out[0][0] - out[1][0])) <= 1e-13

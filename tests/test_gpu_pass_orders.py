"""A workgroup order that was set (the launch otherwise automatic) holds for
two-step passes as well: plain, XCD-contiguous, the fields of a geometry
interleaved, and both.  M_final bit for bit between the orders, and E too (a
field's sums are taken in the order of its own workgroups)."""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_workgroup_orders_of_passes(prec):
    import torch
    import paper_1907_00908_amd as btl
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    btl.load_library()
    # a ragged batch: fields that share a geometry, and fields that do not
    cfg = w.make_config("cfg3b", n=56, K=5, n_q=6)
    out = []
    for xcd in (-1, 0, 1, 2, 3):
        print(f"GPU pass order {xcd} {prec}", flush=True)
        sim = btl.Simulator(cfg["geoms"], cfg["bc"], prec, launch=(-1, 0, xcd))
        try:
            E, M = sim.forward(cfg["dt"], cfg["D"], cfg["T2"], cfg["kappa"], cfg["f"], cfg["gG0"],
                               cfg["q_geom"], want_M=True)
            assert btl.btl_get_forward_passes(sim._h) == (2, 1)
            torch.cuda.synchronize()
            out.append((E.cpu().numpy(), np.concatenate([m.cpu().numpy().ravel() for m in M])))
        finally:
            sim.close()
    for E, M in out[1:]:
        assert np.array_equal(E, out[0][0])
        assert np.array_equal(M, out[0][1])

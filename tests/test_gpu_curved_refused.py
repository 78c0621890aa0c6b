"""A btl_forward_noalloc whose tables of curved links do not fit the buffers
that earlier forwards made is refused and leaves the simulator as it was: the
constants of before still run, on their own tables (the ranges of the refused
tables would reach beyond these).  Bit for bit, since nothing else changes."""
import math

import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("first", [math.inf, 0.0])
def test_refused_tables_leave_the_old_ones(first, prec):
    import torch
    import paper_1907_00908_amd as btl
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    btl.load_library()
    cfg = w.make_config("cfg4", n=(33, 30, 21), K=20, n_q=2, membranes="curved")
    print(f"GPU curved refused after kappa={first} {prec}", flush=True)

    def args(k):
        kappa = np.array([[math.inf, k], [k, math.inf]])
        return cfg["dt"], cfg["D"], cfg["T2"], kappa, cfg["f"], cfg["gG0"], cfg["q_geom"]
    sim = btl.Simulator(cfg["geoms"], cfg["bc"], prec)
    try:
        E0 = sim.forward(*args(first)).cpu().numpy()
        with pytest.raises(btl.BtlError) as ei:
            sim.forward(*args(0.02), noalloc=True)
        assert ei.value.status == btl.BTL_E_UNSUPPORTED
        assert np.array_equal(sim.forward(*args(first)).cpu().numpy(), E0)
        assert np.array_equal(sim.forward(*args(first), noalloc=True).cpu().numpy(), E0)
        E1 = sim.forward(*args(0.02)).cpu().numpy()
        assert np.array_equal(sim.forward(*args(0.02), noalloc=True).cpu().numpy(), E1)
        assert not np.array_equal(E0, E1)
        # room now: the small tables in the larger buffers
        assert np.array_equal(sim.forward(*args(first), noalloc=True).cpu().numpy(), E0)
    finally:
        sim.close()

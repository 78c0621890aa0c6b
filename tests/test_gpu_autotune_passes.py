"""The autotuner's choice holds for later forwards of many steps, so a probe of
one step (or of an odd number) has to let two-step passes compete as they will
run.  Passes take 15 to 20 % less than the best single steps on these lattices,
more than probes differ by: they have to win.  (Each number of steps has a
lattice of its own: choices are remembered by shape.)"""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,K_probe", [((128, 128, 128), 1), ((128, 128, 120), 3)])
def test_odd_probes_let_passes_compete(n, K_probe):
    import torch
    import paper_1907_00908_amd as btl
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    btl.load_library()
    cfg = w.make_config("cfg4", n=n, K=6, n_q=24)
    print(f"GPU autotune {n} probes of {K_probe} steps", flush=True)
    sim = btl.Simulator(cfg["geoms"], cfg["bc"], "f32")
    args = (cfg["dt"], cfg["D"], cfg["T2"], cfg["kappa"], cfg["f"], cfg["gG0"], cfg["q_geom"])
    try:
        E0 = sim.forward(*args).cpu().numpy()
        assert btl.btl_get_forward_passes(sim._h) == (3, 0)
        btl.btl_autotune(sim._h, 0, K_probe, torch.cuda.current_stream().cuda_stream)
        assert btl.btl_get_forward_passes(sim._h) == (3, 0)   # of the caller's forward, not a probe's
        E1 = sim.forward(*args).cpu().numpy()
        assert btl.btl_get_forward_passes(sim._h) == (3, 0)
        assert np.max(np.abs(E0 - E1)) <= 1e-13
    finally:
        sim.close()

"""The automatic launch (short z chunks whose length follows the lattice, the
precision, the membranes and the grid size) against whole columns: M_final bit
for bit (the arithmetic of a site does not depend on its chunk), E to the
rounding of its FP64 sums, which are taken in another order: n terms of size
<= 1 summed with unit roundoff 1.1e-16 differ by at most n 1.1e-16 and, for
the pairwise trees used here, by far less; 1e-13 covers it.  Sizes at the
edges of the rule: fewer layers than a chunk, remainders, one workgroup, and a
btl_forward_noalloc that fits the scratch only as whole columns.
"""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


def _gpu():
    import torch
    import paper_1907_00908_amd as btl
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    btl.load_library()
    return btl, torch


def _run(cfg, prec, launch=None, noalloc=False, scheme=0):
    btl, torch = _gpu()
    sim = btl.Simulator(cfg["geoms"], cfg["bc"], prec, scheme, lattice=cfg.get("lattice", 0),
                        launch=launch)
    try:
        E, M = sim.forward(cfg["dt"], cfg["D"], cfg["T2"], cfg["kappa"], cfg["f"], cfg["gG0"],
                           cfg["q_geom"], want_M=True, noalloc=noalloc)
        torch.cuda.synchronize()
        return E.cpu().numpy(), np.concatenate([m.cpu().numpy().ravel() for m in M])
    finally:
        sim.close()


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("name,kw,scheme", [
    ("cfg4", dict(n=(16, 14, 1), n_q=1), 0), ("cfg4", dict(n=(17, 15, 2), n_q=2), 0),
    ("cfg4", dict(n=(33, 9, 4), n_q=3), 0), ("cfg4", dict(n=(96, 88, 31), n_q=7), 0),
    ("cfg4", dict(n=(48, 40, 23), n_q=4), 1), ("cfg2", dict(n=(40, 36, 29)), 0),
    ("cfg2", dict(n=(32, 20, 17), membranes="positions"), 0),
    ("cfg2", dict(n=(24, 20, 15), membranes="curved"), 0), ("cfg2d", dict(n=100, n_q=9), 0)])
def test_automatic_chunks_equal_whole_columns(name, kw, scheme, prec):
    kw = dict(kw)
    cfg = w.make_config(name, K=9, **kw)
    print(f"GPU chunks {name} {kw} scheme={scheme} {prec}", flush=True)
    whole = (4 if name == "cfg2d" else 3, 0, 0)
    E0, M0 = _run(cfg, prec, launch=whole, scheme=scheme)
    E1, M1 = _run(cfg, prec, scheme=scheme)
    assert np.array_equal(M0, M1)
    assert np.max(np.abs(E0 - E1)) <= 1e-13


def test_noalloc_falls_back_to_whole_columns():
    # 133.0 MB of populations leave 1.2 MB of the 134.2 MB scratch: with the
    # phase tables (0.2 MB) the signal partials of 3-site chunks (3.2 MB) do
    # not fit, those of whole columns do
    cfg = w.make_config("cfg1", n=(64, 64, 290), K=5)
    print("GPU noalloc at the scratch limit", flush=True)
    E0, M0 = _run(cfg, "f32")
    E1, M1 = _run(cfg, "f32", noalloc=True)
    assert np.array_equal(M0, M1)
    assert np.max(np.abs(E0 - E1)) <= 1e-13

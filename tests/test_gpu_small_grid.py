"""Grids of at most 2048 workgroups take a form of the step kernel that loads
the first site ahead of its tables; larger ones do not.  The arithmetic of a
site is the same in both, so a weighting gives M_final bit for bit alone and
among as many others as pass the limit, and E to the rounding of the per-block
FP64 sums (same blocks, same order inside a block; the order over blocks may
differ: n terms of size <= 1 and pairwise trees, 1e-13 covers it).  Lattices at
the edges: planes that do not fill a tile, one site a thread, an odd and an
even number of sites, a column as long as a workgroup and one longer.
"""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu


def _run(cfg, prec, launch):
    import torch
    import paper_1907_00908_amd as btl
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    btl.load_library()
    sim = btl.Simulator(cfg["geoms"], cfg["bc"], prec, 0, lattice=cfg.get("lattice", 0),
                        launch=launch)
    try:
        E, M = sim.forward(cfg["dt"], cfg["D"], cfg["T2"], cfg["kappa"], cfg["f"], cfg["gG0"],
                           cfg["q_geom"], want_M=True)
        torch.cuda.synchronize()
        return E.cpu().numpy(), [m.cpu().numpy() for m in M]
    finally:
        sim.close()


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("name,kw,launch,n_q", [
    ("cfg4", dict(n=(33, 9, 5)), (3, 1, 0), 90), ("cfg4", dict(n=(33, 9, 5)), (3, 2, 1), 150),
    ("cfg4", dict(n=(20, 17, 7)), (5, 3, 0), 400), ("cfg4", dict(n=(7, 5, 6)), (0, 6, 0), 1100),
    ("cfg4", dict(n=(5, 3, 256)), (1, 256, 0), 2100),
    ("cfg4", dict(n=(5, 3, 300)), (1, 300, 0), 2100), ("cfg2d", dict(n=37), (4, 2, 0), 110)])
def test_alone_equals_in_a_long_grid(name, kw, launch, n_q, prec):
    big = w.make_config(name, K=5, n_q=n_q, **kw)
    print(f"GPU small grid {name} {kw} {launch} x {n_q} {prec}", flush=True)
    E0, M0 = _run(big, prec, launch)
    for q in (0, n_q - 1):
        one = dict(big, gG0=big["gG0"][q:q + 1])
        one["q_geom"] = big["q_geom"][q:q + 1]
        E1, M1 = _run(one, prec, launch)
        assert np.array_equal(M0[q], M1[0])
        assert np.max(np.abs(E0[q] - E1[0])) <= 1e-13

"""Half-link membranes that let little or nothing through, between a phase
without relaxation and one that decays by 18 orders of magnitude: the faint
side then holds what the membrane transmits alone, so a share t held to an
absolute 1e-16 instead of its own precision (own + t (in - own)) shows there.

M_final against the FP64 oracle, relative at every site.  A step multiplies a
population by at most eight rounded factors and sums, so 40 steps keep FP64
storage within 40 x 8 x 1.1e-16 = 3.6e-14 (1e-12 used: the oracle rounds too,
in another order) and FP32 storage, rounded once a step, within 40 x 6e-8 =
2.4e-6 (1e-5 used).  Single steps (a set launch, short and long grids) and two
steps per pass (the automatic launch on these 1020 and 780 tiles), both
lattices.  Permeable membranes on wide disks are left to the other parity
tests: M then changes its sign from site to site far inside, and next to such a
site it has no relative precision in either code (100^2, kappa 0.02: a change
of D by 2e-16 moves the oracle's M by 9e-13).
"""
import math

import numpy as np
import pytest

import oracle
import workloads as w

pytestmark = pytest.mark.gpu


def _check(cfg, kappa, prec, launch, n_q):
    import torch
    import paper_1907_00908_amd as btl
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    btl.load_library()
    K = 40
    cfg["kappa"] = np.array([[math.inf, kappa], [kappa, math.inf]])
    cfg["T2"] = np.array([math.inf, K * cfg["dt"] / (18.0 * math.log(10.0))])
    cfg["f"] = np.ones(K)
    cfg["gG0"] = np.zeros((n_q, 3))
    cfg["q_geom"] = np.zeros(n_q, np.int32)
    sim = btl.Simulator(cfg["geoms"], cfg["bc"], prec, lattice=cfg.get("lattice", 0), launch=launch)
    try:
        _, M = sim.forward(cfg["dt"], cfg["D"], cfg["T2"], cfg["kappa"], cfg["f"], cfg["gG0"],
                           cfg["q_geom"], want_M=True)
        torch.cuda.synchronize()
        M = [M[q].cpu().numpy() for q in (0, n_q - 1)]
    finally:
        sim.close()
    _, Mo = oracle.simulate_config(cfg, q=[0], threads=8, want_M=True)
    rtol = 1e-12 if prec == "f64" else 1e-5
    for m in M:
        err = np.max(np.abs(m - Mo[0]) / np.abs(Mo[0]))
        assert err <= rtol, err


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("kappa", [0.0, 1e-13, 0.02])
@pytest.mark.parametrize("launch,n_q", [((1, 4, 0), 1), ((1, 1, 0), 60), (None, 170)])
def test_small_shares_d3q7(launch, n_q, kappa, prec):
    cfg = w.make_config("cfg2", n=(24, 22, 18))
    cfg["bc"] = [0, 0, 0]
    print(f"GPU membrane share D3Q7 {launch} x {n_q} kappa={kappa} {prec}", flush=True)
    _check(cfg, kappa, prec, launch, n_q)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("kappa", [0.0, 1e-13])
@pytest.mark.parametrize("launch,n_q", [((4, 4, 0), 1), (None, 60)])
def test_small_shares_d2q5(launch, n_q, kappa, prec):
    cfg = w.make_config("cfg2d", n=100)
    print(f"GPU membrane share D2Q5 {launch} x {n_q} kappa={kappa} {prec}", flush=True)
    _check(cfg, kappa, prec, launch, n_q)

"""Two steps per pass (k_pair, the default of untuned hybrid forwards on
half-link membranes) against single steps (a launch that was set): M_final bit
for bit, since the state between the two steps is rounded as a stored one and
a site's arithmetic is the same; E to the rounding of FP64 sums taken in
another order (1e-13, as in test_gpu_chunks).  Sizes where the tiles, the ring
columns and the z walk can go wrong: fewer sites than a tile, remainders along
every axis, single layers, more than one z chunk, wrapped rings of two or
three sites, mirrored faces with one to four fields, ragged batches, odd and
even numbers of steps, more steps than one phase table holds.
"""
import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu

P, R = 0, 1   # periodic, mirrored


def _gpu():
    import torch
    import paper_1907_00908_amd as btl
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    btl.load_library()
    return btl, torch


def _forward(cfg, prec, launch=None, ckpt=0, noalloc=False):
    btl, torch = _gpu()
    sim = btl.Simulator(cfg["geoms"], cfg["bc"], prec, lattice=cfg.get("lattice", 0), launch=launch)
    try:
        E, M = sim.forward(cfg["dt"], cfg["D"], cfg["T2"], cfg["kappa"], cfg["f"], cfg["gG0"],
                           cfg["q_geom"], want_M=True, ckpt_every=ckpt, noalloc=noalloc)
        torch.cuda.synchronize()
        return E.cpu().numpy(), np.concatenate([m.cpu().numpy().ravel() for m in M])
    finally:
        sim.close()


def _check(cfg, prec, **kw):
    single = (4 if cfg.get("lattice", 0) else 1, 4, 0)
    E0, M0 = _forward(cfg, prec, launch=single)
    E1, M1 = _forward(cfg, prec, **kw)
    assert np.array_equal(M0, M1), np.max(np.abs(M0 - M1))
    assert np.max(np.abs(E0 - E1)) <= 1e-13


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,bc,K", [
    ((2, 2, 1), (P, P, P), 4), ((3, 2, 2), (R, P, R), 5), ((16, 14, 5), (P, P, P), 7),
    ((33, 9, 4), (R, R, R), 6), ((40, 21, 70), (R, P, R), 5), ((50, 47, 13), (P, R, P), 8),
    ((70, 19, 66), (P, P, R), 4), ((96, 88, 31), (R, R, P), 3), ((131, 37, 34), (R, R, R), 5),
    ((300, 7, 35), (P, P, P), 4), ((24, 20, 12), (R, P, P), 67)])
def test_two_steps_per_pass_d3q7(n, bc, K, prec):
    cfg = w.make_config("cfg2" if min(n) > 3 else "cfg1", n=n, K=K)
    cfg["bc"] = list(bc)
    g = np.array([[0.7, -0.4, 0.59], [0.0, 0.8, 0.6], [0.5, 0.0, 0.0]]) * 0.05
    cfg["gG0"], cfg["q_geom"] = g, np.zeros(3, np.int32)
    print(f"GPU pair {n} {bc} K={K} {prec}", flush=True)
    _check(cfg, prec)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,bc,K", [((40, 40, 1), (P, P, P), 9), ((515, 33, 1), (R, R, P), 6),
                                    ((128, 128, 1), (R, P, P), 5), ((254, 70, 1), (P, R, P), 4)])
def test_two_steps_per_pass_d2q5(n, bc, K, prec):
    cfg = w.make_config("cfg2d", n=128, K=K, n_q=4)
    g = cfg["geoms"][0]
    reps = (-(-n[0] // 128), -(-n[1] // 128))
    comp = np.tile(g.comp, (1, reps[1], reps[0]))[:, :n[1], :n[0]]
    g.comp = np.ascontiguousarray(comp)
    cfg["bc"] = list(bc)
    print(f"GPU pair D2Q5 {n} {bc} K={K} {prec}", flush=True)
    _check(cfg, prec)


def test_two_steps_per_pass_ragged_batch():
    cfg = w.make_config("cfg3b", n=40, K=6, n_q=2)
    print("GPU pair ragged", flush=True)
    _check(cfg, "f32")


@pytest.mark.parametrize("ckpt", [4, 5, 100])
def test_two_steps_per_pass_with_a_tape(ckpt):
    cfg = w.make_config("cfg2", n=(24, 22, 18), K=13, n_q=2)
    print(f"GPU pair with a tape, every {ckpt}", flush=True)
    _check(cfg, "f32", ckpt=ckpt)


def test_two_steps_per_pass_noalloc():
    cfg = w.make_config("cfg2", n=(24, 22, 18), K=13, n_q=2)
    print("GPU pair without allocation", flush=True)
    _check(cfg, "f32", noalloc=True)

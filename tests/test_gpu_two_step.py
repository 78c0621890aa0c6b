"""Two steps per pass (k_pair) against single steps, on grids that really take
passes: the automatic launch does from 700 workgroups on (FP32 D3Q7: 1000),
each case has enough q-samples for that, and btl_get_forward_passes has to say
so.

M_final bit for bit, since the state between the two steps is rounded as a
stored one and a site's arithmetic is the same; E to the rounding of FP64 sums
taken in another order (n terms of size <= 1 with unit roundoff 1.1e-16,
pairwise trees: 1e-13 covers it); gradients bit for bit where both tapes have
the adjoint's launch in common.  Sizes where the tiles, the ring columns and
the z walk can go wrong: fewer sites than a tile, remainders along every axis,
single layers, short and long z chunks, wrapped rings of two or three sites,
mirrored faces with one to four fields, ragged batches, odd and even numbers of
steps, more steps than one phase table holds, tapes, q-waves, graphs, the
unallocating entry, links whose membrane lets everything through.
"""
import math

import numpy as np
import pytest

import workloads as w

pytestmark = pytest.mark.gpu

P, R = 0, 1   # periodic, mirrored
INF = math.inf


def _gpu():
    import torch
    import paper_1907_00908_amd as btl
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    btl.load_library()
    return btl, torch


def _forward(cfg, prec, passes, launch=None, ckpt=0, noalloc=False, dLdE=None, **options):
    btl, torch = _gpu()
    sim = btl.Simulator(cfg["geoms"], cfg["bc"], prec, lattice=cfg.get("lattice", 0), launch=launch,
                        **options)
    try:
        E, M = sim.forward(cfg["dt"], cfg["D"], cfg["T2"], cfg["kappa"], cfg["f"], cfg["gG0"],
                           cfg["q_geom"], want_M=True, ckpt_every=ckpt, noalloc=noalloc)
        assert btl.btl_get_forward_passes(sim._h) == passes
        grads = []
        if dLdE is not None:
            g = torch.as_tensor(dLdE, dtype=torch.float64, device="cuda")
            grads = [x.cpu().numpy() for x in sim.backward(g)]
        torch.cuda.synchronize()
        return E.cpu().numpy(), np.concatenate([m.cpu().numpy().ravel() for m in M]), grads
    finally:
        sim.close()


def _check(cfg, prec, single=None, passes=None, **kw):
    K = len(cfg["f"])
    single = single or ((4 if cfg.get("lattice", 0) else 1), 4, 0)
    E0, M0, g0 = _forward(cfg, prec, (0, K), launch=single, ckpt=kw.get("ckpt", 0),
                          dLdE=kw.get("dLdE"))
    E1, M1, g1 = _forward(cfg, prec, passes or (K // 2, K % 2), **kw)
    assert np.array_equal(M0, M1), np.max(np.abs(M0 - M1))
    assert np.max(np.abs(E0 - E1)) <= 1e-13
    for a, b in zip(g0, g1):
        assert np.array_equal(a, b)


def _d3q7(n, bc, K, reps):
    """reps times a general gradient, one in the y-z plane and one along x."""
    cfg = w.make_config("cfg2" if min(n) > 3 else "cfg1", n=n, K=K)
    cfg["bc"] = list(bc)
    g = np.array([[0.7, -0.4, 0.59], [0.0, 0.8, 0.6], [0.5, 0.0, 0.0]]) * 0.05
    cfg["gG0"] = np.concatenate([g * s for s in np.linspace(0.5, 1.0, reps)])
    cfg["q_geom"] = np.zeros(3 * reps, np.int32)
    return cfg


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,bc,K,reps", [
    ((2, 2, 1), (P, P, P), 4, 340), ((3, 2, 2), (R, P, R), 5, 150), ((16, 14, 5), (P, P, P), 7, 340),
    ((33, 9, 4), (R, R, R), 6, 150), ((40, 21, 70), (R, P, R), 5, 6), ((50, 47, 13), (P, R, P), 8, 15),
    ((70, 19, 66), (P, P, R), 4, 6), ((96, 88, 31), (R, R, P), 3, 2), ((131, 37, 34), (R, R, R), 5, 2),
    ((300, 7, 35), (P, P, P), 4, 12), ((24, 20, 12), (R, P, P), 67, 65), ((6, 5, 130), (P, P, R), 5, 300),
    ((6, 5, 70), (R, P, P), 4, 450), ((8, 7, 40), (P, R, R), 2, 300)])
def test_d3q7(n, bc, K, reps, prec):
    print(f"GPU two-step {n} {bc} K={K} x {reps} {prec}", flush=True)
    _check(_d3q7(n, bc, K, reps), prec)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n,bc,K,n_q", [
    ((40, 40, 1), (P, P, P), 9, 150), ((515, 33, 1), (R, R, P), 6, 25),
    ((128, 128, 1), (R, P, P), 5, 24), ((254, 70, 1), (P, R, P), 4, 45)])
def test_d2q5(n, bc, K, n_q, prec):
    cfg = w.make_config("cfg2d", n=128, K=K, n_q=n_q)
    g = cfg["geoms"][0]
    reps = (-(-n[0] // 128), -(-n[1] // 128))
    comp = np.tile(g.comp, (1, reps[1], reps[0]))[:, :n[1], :n[0]]
    g.comp = np.ascontiguousarray(comp)
    cfg["bc"] = list(bc)
    print(f"GPU two-step D2Q5 {n} {bc} K={K} x {n_q} {prec}", flush=True)
    _check(cfg, prec)


def test_ragged_batch():
    cfg = w.make_config("cfg3b", n=40, K=6, n_q=6)
    print("GPU two-step ragged", flush=True)
    _check(cfg, "f32")


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_permeable_and_open_links(prec):
    # three phases, one pair of which has no membrane between its compartments
    cfg = w.make_config("cfg3a", n=(40, 36, 34), K=6, n_q=52)
    cfg["kappa"][0, 2] = cfg["kappa"][2, 0] = INF
    print(f"GPU two-step open links {prec}", flush=True)
    _check(cfg, prec)


@pytest.mark.parametrize("ckpt", [4, 5, 100])
def test_with_a_tape(ckpt):
    # rows (shape 5) are the automatic tile of these lattices, so that both
    # tapes have the same adjoint launch; an odd interval takes single steps
    cfg = w.make_config("cfg4", n=(37, 35, 18), K=13, n_q=90)
    rng = np.random.default_rng(5)
    print(f"GPU two-step with a tape, every {ckpt}", flush=True)
    _check(cfg, "f32", single=(5, 4, 0), passes=(0, 13) if ckpt == 5 else (6, 1), ckpt=ckpt,
           dLdE=rng.standard_normal((90, 14, 2)))


def test_q_waves():
    # a budget of half the states: groups of 361 and 359 q-samples
    cfg = _d3q7((16, 14, 24), (P, P, P), 5, 240)
    one = 7 * 16 * 14 * 24 * 8
    print("GPU two-step q-waves", flush=True)
    _check(cfg, "f32", passes=(4, 2), mem_budget=2 * one * 361)


@pytest.mark.parametrize("graphs", [False, True])
def test_many_steps(graphs):
    cfg = _d3q7((16, 14, 17), (P, P, P), 35, 115)
    print(f"GPU two-step 35 steps, graphs {graphs}", flush=True)
    _check(cfg, "f32", graphs=graphs)


@pytest.mark.parametrize("n,K,reps", [((5, 4, 9), 6, 170), ((12, 10, 9), 7, 180)])
def test_noalloc(n, K, reps):
    print(f"GPU two-step without allocation {n}", flush=True)
    _check(_d3q7(n, (P, P, P), K, reps), "f32", noalloc=True)


def test_set_launches_take_single_steps():
    cfg = _d3q7((16, 14, 5), (P, P, P), 4, 340)
    for launch in [(0, 2, 0), (-1, 3, 1)]:
        _forward(cfg, "f32", (0, 4), launch=launch)
    cfg["gG0"], cfg["q_geom"] = cfg["gG0"][:30], cfg["q_geom"][:30]
    _forward(cfg, "f32", (0, 4))   # 30 workgroups

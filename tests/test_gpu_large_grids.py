"""Batches of so many fields that short z chunks (or a wave per sum of the
gradients) would pass the 2^32 threads of a launch: columns are cut less, and
the sums are taken in several launches.  Signals against the field alone (FP64
sums of terms <= 1 in another order: 1e-13), gradients bit for bit against a
tape of short segments (the same sums over the same states)."""
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


def _cfg(n, K, n_q):
    cfg = w.make_config("cfg1", n=n, K=K)
    cfg["gG0"] = np.array([0.3, -0.2, 0.59]) * np.linspace(0.01, 0.05, n_q)[:, None]
    cfg["q_geom"] = np.zeros(n_q, np.int32)
    return cfg


def test_chunks_of_very_many_columns():
    # 49200 fields of 2 x 2 x 1024, 16.8 million chunks of three sites; the
    # last of three steps goes by itself
    btl, torch = _gpu()
    n_q = 49200
    cfg = _cfg((2, 2, 1024), 3, n_q)
    print("GPU 49200 columns", flush=True)
    sim = btl.Simulator(cfg["geoms"], cfg["bc"], "f32")

    def run(sel):
        return sim.forward(cfg["dt"], cfg["D"], cfg["T2"], cfg["kappa"], cfg["f"],
                           cfg["gG0"][sel], cfg["q_geom"][sel]).cpu().numpy()
    try:
        E = run(slice(None))
        for q in (0, 24600, n_q - 1):
            assert np.max(np.abs(run(slice(q, q + 1))[0] - E[q])) <= 1e-13
    finally:
        sim.close()
        torch.cuda.empty_cache()


def test_gradient_sums_of_very_many_steps_and_fields():
    # one phase: 5 accumulators of 14000 fields in 1000 steps are 70 million
    # sums, a wave each
    btl, torch = _gpu()
    n_q, K = 14000, 1000
    cfg = _cfg((3, 3, 2), K, n_q)
    rng = np.random.default_rng(3)
    g = torch.as_tensor(rng.standard_normal((n_q, K + 1, 2)), device="cuda")
    out = []
    for ckpt in (1000, 100):
        print(f"GPU 14000 fields, 1000 steps, segments of {ckpt}", flush=True)
        sim = btl.Simulator(cfg["geoms"], cfg["bc"], "f32")
        try:
            sim.forward(cfg["dt"], cfg["D"], cfg["T2"], cfg["kappa"], cfg["f"], cfg["gG0"],
                        cfg["q_geom"], ckpt_every=ckpt)
            out.append([x.cpu().numpy() for x in sim.backward(g)])
            assert btl.btl_get_backward_stats(sim._h)[2] == 0   # a uniform tape
        finally:
            sim.close()
    for a, b in zip(*out):
        assert np.all(np.isfinite(a)) and np.array_equal(a, b)

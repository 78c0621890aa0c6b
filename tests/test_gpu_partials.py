"""Signal partial sums: held for as many steps as 64 MiB take, and in the
unallocating entry for as many as its scratch has room for; block tables only
for launches that are made.  How often the signals are summed does not change
a step's sums: E and M_final bit for bit against a small batch of the same
launch, and for passes the bounds of the other comparisons (1e-13 on E, sums of
FP64 terms <= 1 in another order)."""
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
    cfg = w.make_config("cfg4" if min(n) > 3 else "cfg1", n=n, K=K)
    cfg["bc"] = [0, 0, 0]
    g = np.array([0.7, -0.4, 0.59]) * 0.05
    cfg["gG0"] = g * np.linspace(0.5, 1.0, n_q)[:, None]
    cfg["q_geom"] = np.zeros(n_q, np.int32)
    return cfg


def _args(cfg, sel=slice(None)):
    return (cfg["dt"], cfg["D"], cfg["T2"], cfg["kappa"], cfg["f"], cfg["gG0"][sel],
            cfg["q_geom"][sel])


@pytest.mark.parametrize("scheme,passes", [(0, (1, 0)), (1, (0, 2))])
def test_memory_beside_the_states(scheme, passes):
    # 6000 fields of 16 x 16 x 48: two states of 4.1 GB, phase tables of 32
    # steps, the signal, 64 MiB of partial sums; 48 MiB for the small tables
    # and the allocator's granularity
    btl, torch = _gpu()
    n_q, n, K = 6000, (16, 16, 48), 2
    cfg = _cfg(n, K, n_q)
    print(f"GPU partial sums, memory, scheme {scheme}", flush=True)
    sim = btl.Simulator(cfg["geoms"], cfg["bc"], "f32", scheme)
    try:
        torch.cuda.synchronize()
        free0 = torch.cuda.mem_get_info()[0]
        E = sim.forward(*_args(cfg))
        torch.cuda.synchronize()
        used = free0 - torch.cuda.mem_get_info()[0]
        assert btl.btl_get_forward_passes(sim._h) == passes
        states = 2 * n_q * 7 * n[0] * n[1] * n[2] * 8
        tables = n_q * (sum(n) + 6) * (32 * 16 + 4)
        assert used <= states + tables + (64 << 20) + (48 << 20), (used - states - tables) / 2**20
        assert E.shape == (n_q, K + 1)
    finally:
        sim.close()


def test_single_steps_with_few_slots():
    # 96000 workgroups: partial sums of 8 steps at a time
    btl, torch = _gpu()
    cfg = _cfg((16, 16, 48), 35, 6000)
    print("GPU partial sums of single steps", flush=True)
    sim = btl.Simulator(cfg["geoms"], cfg["bc"], "f32", launch=(2, 3, 0))
    try:
        E = sim.forward(*_args(cfg)).cpu().numpy()
        for q in (0, 3000, 5999):
            one = sim.forward(*_args(cfg, slice(q, q + 1))).cpu().numpy()
            assert np.array_equal(E[q], one[0])
    finally:
        sim.close()


def test_passes_with_few_slots():
    # 140000 workgroups either way: passes sum every 16 steps, single steps
    # every 4
    btl, torch = _gpu()
    cfg = _cfg((2, 2, 1), 35, 140000)
    out = []
    print("GPU partial sums of passes", flush=True)
    for launch, passes in ((None, (17, 1)), ((0, 1, 0), (0, 35))):
        sim = btl.Simulator(cfg["geoms"], cfg["bc"], "f32", launch=launch, graphs=False)
        try:
            E, M = sim.forward(*_args(cfg), want_M=True)
            torch.cuda.synchronize()
            assert btl.btl_get_forward_passes(sim._h) == passes
            out.append((E.cpu().numpy(), np.concatenate([m.cpu().numpy().ravel() for m in M[::7]])))
        finally:
            sim.close()
    assert np.array_equal(out[0][1], out[1][1])
    assert np.max(np.abs(out[0][0] - out[1][0])) <= 1e-13


@pytest.mark.parametrize("K", [6, 7])
def test_noalloc_near_the_scratch_limit_keeps_passes(K):
    # 930 fields of 12 x 10 x 9: 112.5 MB of states and 17.7 MB of phase tables
    # in 134.2 MB; the partial sums of 32 single steps would be 5.7 MB
    btl, torch = _gpu()
    cfg = _cfg((12, 10, 9), K, 930)
    print(f"GPU partial sums at the scratch limit K={K}", flush=True)
    out = []
    for noalloc in (False, True):
        sim = btl.Simulator(cfg["geoms"], cfg["bc"], "f32")
        try:
            E, M = sim.forward(*_args(cfg), want_M=True, noalloc=noalloc)
            torch.cuda.synchronize()
            assert btl.btl_get_forward_passes(sim._h) == (K // 2, K % 2)
            out.append((E.cpu().numpy(), np.concatenate([m.cpu().numpy().ravel() for m in M])))
        finally:
            sim.close()
    assert np.array_equal(out[0][1], out[1][1])
    assert np.array_equal(out[0][0], out[1][0])

"""Curved links are evaluated in runs: up to 256 links whose terms read at most
as many 128-byte lines as LDS holds, with the periodic factors of a term looked
up by a code.  Parity with the FP64 oracle, with the tolerances of the other
parity tests (FP64 storage |dE| <= 1e-12 |E| + 1e-14, FP32 |dE| <= 1e-5 |E|
where |E| >= 1e-2 and 1e-7 below), where that can go wrong: axes of two
sites (terms beyond their faces), a single run with idle waves, packings
whose runs end by lines and by links, and one and several groups of fields,
the last one not full.
"""
import numpy as np
import pytest

import workloads as w

from .test_gpu_curved import _both, _strong
from .test_gpu_parity import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("name,kw,n_q", [
    ("cfg4", dict(n=(20, 2, 6)), 2), ("cfg4", dict(n=(2, 20, 6)), 1),
    ("cfg4", dict(n=(17, 15, 1)), 3), ("cfg4", dict(n=(33, 30, 21)), 13),
    ("cfg3a", dict(n=44), 5)])
def test_link_runs_match_the_oracle(name, kw, n_q, prec):
    cfg = w.make_config(name, K=24, membranes="curved", **kw)
    q = np.arange(n_q) % len(cfg["gG0"])
    cfg["gG0"] = cfg["gG0"][q] * np.linspace(0.5, 1.5, n_q)[:, None]
    cfg["q_geom"] = cfg["q_geom"][q]
    cfg = _strong(cfg)
    Eg, Mg, Eo, Mo = _both(cfg, prec, want_M=True)
    _check(Eg, Eo, prec, f"{name} {kw}")
    for k in range(n_q):
        _check(Mg[k], Mo[k], prec, f"{name} {kw} M_final q={k}")

"""The walk's rounds and calm stretches at their edges (-m gpu): step caps and
roulette around the 32 steps a wave takes between looks at them, photons that
start, stay or end within the margin of a wall, thresholds of a round that
meet one photon, one wave and a remainder."""
import numpy as np
import pytest

import workloads as W
from _helpers import assert_matched_scalars, gpu_run, oracle_rec, trajectory_match
from oracle import walk as owalk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(max_steps=1, tau=3.0), dict(max_steps=31, tau=12.0), dict(max_steps=32, tau=12.0),
    dict(max_steps=33, tau=12.0), dict(max_steps=65, tau=16.0, albedo=1.0),
    dict(tau=10.0, albedo=0.9, roulette_w=0.03, roulette_p=0.5),      # roulette from about step 32 on
    dict(tau=10.0, albedo=0.0, roulette_w=0.0),                       # weight 0, never killed
    dict(tau=10.0, albedo=0.7, roulette_w=2.0, roulette_p=0.9),       # every weight below the threshold
    dict(tau=2e-4, size_mm=(10.0, 10.0, 1e-3)),                       # a thin slab
    dict(tau=60.0, n_photons=2000),                                   # many steps, many of them by the entry face
    dict(tau=2.0, size_mm=(0.02, 50.0, 10.0), src_pos_mm=(0.01, 25.0, 0.0)),   # a narrow channel: mostly walls
    dict(tau=4.0, src_pos_mm=(0.0, 10.0, 0.0), src_dir=(0.2, -0.4, 0.8)),      # from an edge
    dict(tau=3.0, n_photons=1), dict(tau=3.0, n_photons=63), dict(tau=3.0, n_photons=65),
], ids=str)
def test_rounds_match_the_oracle(cuda_device, kw):
    kw = dict(kw)
    w = W.TINY.replace(**{"n_photons": 20000, "side_px": 32, "trans_px": 32, **kw})
    g = gpu_run(w, records=True, fix64=True)
    o = owalk.Walk(w).run(records=True)
    orec = oracle_rec(o)
    ok = trajectory_match(g["rec"], orec, box=max(w.size_mm))
    # FP32 transport may part from the oracle's at a wall or a draw, at a rate
    # per step that leaves 99.9 % of photons of the usual few steps alike.
    steps = max(1.0, float(np.mean(orec["steps"])) / 10.0)
    assert 1.0 - ok.mean() <= max(1e-3 * steps, 0.0 if w.n_photons > 1000 else 1.5 / w.n_photons), (kw, ok.mean())
    assert_matched_scalars(g["scalars"], g["rec"], o.scalars, orec, ok)
    # The kernels without records walk the same photons, bit for bit.
    p = gpu_run(w, fix64=True)
    for name in ("side", "trans", "side_w2", "trans_w2", "scalars"):
        assert np.array_equal(p[name], g[name]), name

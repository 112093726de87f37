"""Exits past the end of their range's region of the exit log (-m gpu): taken by
the block's cache, by image copy 0, or, for many photons in small images, by a
copy per XCD.  Fixed-point sums: every image and scalar equals the atomic
path's bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

SMALL, MID, MANY = 300_000, 8_000_000, 1 << 24    # SMALL fits every log, MID not; MANY with at most 2^17 pixels: a copy per XCD


@pytest.fixture(scope="module")
def mc():
    import paper_2507_23189_amd as m
    m.lib()
    return m


@pytest.fixture(scope="module")
def table(mc, cuda_device):
    return mc.mie_table_build(mc.args_from_workload(W.TINY)[0], cuda_device)


def _run(mc, table, n, px, flags, log_photons, times=1):
    import torch
    w = W.TINY.replace(tau=1.0, n_photons=n, side_px=px, trans_px=px)
    _, med, src, geo, det, run = mc.args_from_workload(w, table, flags=flags)
    t = mc.Tally.alloc(det, "cuda", sigma=bool(flags & mc.MC_SIGMA), fix64=bool(flags & mc.MC_FIX64),
                       log_photons=log_photons)
    for img in (t.side, t.trans, t.scalars):
        img.zero_()
    for _ in range(times):
        mc.mc_simulate(med, src, geo, det, run, t)
    torch.cuda.synchronize()
    out = {k: getattr(t, k).cpu().numpy() for k in ("side", "trans", "scalars", "side_w2", "trans_w2")
           if getattr(t, k) is not None}
    return out, int(t.workspace[21].item())


@pytest.mark.parametrize("n, px, log_photons", [
    (SMALL, 16, SMALL // 4), (SMALL, 64, 0), (SMALL, 300, SMALL // 8),        # (every region holds 64 exits or more)
    (MID, 16, MID // 4), (MID, 64, 0), (MID, 300, MID // 8),
    (MANY - 1, 64, MANY // 8), (MANY, 64, MANY), (MANY, 256, MANY // 8), (MANY, 257, MANY // 8),
], ids=str)
@pytest.mark.parametrize("sigma", [False, True], ids=["", "sigma"])
def test_overflow_equals_the_atomic_path(mc, table, cuda_device, n, px, log_photons, sigma):
    flags = mc.MC_FIX64 | (mc.MC_SIGMA if sigma else 0)
    got, full = _run(mc, table, n, px, flags | mc.MC_EXIT_LOG, log_photons)
    ref, none = _run(mc, table, n, px, flags, None)
    assert (full > 0) == (n > SMALL) and none == 0
    for k in ref:
        assert np.array_equal(got[k], ref[k]), k


@pytest.mark.parametrize("n", [SMALL, MID, MANY])
def test_overflow_of_added_launches(mc, table, cuda_device, n):
    one, _ = _run(mc, table, n, 32, mc.MC_FIX64, None)
    two, full = _run(mc, table, n, 32, mc.MC_FIX64 | mc.MC_EXIT_LOG | mc.MC_ACCUMULATE, n // 8, times=2)
    assert (full > 0) == (n > SMALL)
    for k in one:
        assert np.array_equal(two[k], 2 * one[k]), k

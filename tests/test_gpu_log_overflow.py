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


@pytest.mark.parametrize("shape", [(37, 23, 61, 19), (1, 1, 1, 1), (5, 300, 700, 3), (512, 512, 1024, 1024)], ids=str)
@pytest.mark.parametrize("n, grid", [(1 << 20, 0), ((1 << 20) + 1, 0), (1 << 19, 0), ((1 << 19) + 1, 0), (200_000, 300),
                                     (200_000, 2)], ids=str)
def test_few_photons_with_and_without_the_log(mc, table, cuda_device, shape, n, grid):
    """Around the counts up to which a launch takes no log, and one or two image
    copies: the sums of a log that the caller's grid asks for."""
    import torch
    w = W.TINY.replace(tau=2.0, n_photons=n, side_px=16, trans_px=16)
    out = []
    for flags, blocks in ((mc.MC_EXIT_LOG, grid), (mc.MC_EXIT_LOG, 256), (0, grid)):
        _, med, src, geo, det, run = mc.args_from_workload(w, table, flags=flags | mc.MC_FIX64 | mc.MC_SIGMA)
        det.side_nx, det.side_ny, det.trans_nx, det.trans_ny = shape
        run.grid_blocks = blocks
        t = mc.Tally.alloc(det, "cuda", sigma=True, fix64=True, log_photons=n)
        mc.mc_simulate(med, src, geo, det, run, t)
        torch.cuda.synchronize()
        out.append([getattr(t, k).cpu().numpy() for k in ("side", "trans", "scalars", "side_w2", "trans_w2")])
    for other in out[1:]:
        for x, y in zip(out[0], other):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("n", [1 << 12, 1 << 13, 1 << 14], ids=str)
def test_few_photons_of_a_batch(mc, table, cuda_device, n):
    """64 media of n photons: one copy, two, and all of them (or the log)."""
    import torch
    _, _, src, geo, det, run = mc.args_from_workload(W.TINY.replace(side_px=16, trans_px=16), table, flags=mc.MC_FIX64)
    out = []
    for flags, blocks, extra in ((0, 0, 0), (mc.MC_EXIT_LOG, 0, 0), (mc.MC_EXIT_LOG, 256, 0), (0, 0, 1)):
        det.flags, run.grid_blocks = mc.MC_FIX64 | flags, blocks
        items = [mc.BatchItem(tau=0.1 * (i + 1), albedo=0.9999, inv_cdf=table.inv_cdf.data_ptr(),
                              n_photons=n + (extra if i == 63 else 0), instance=i) for i in range(64)]
        t = mc.Tally.alloc_batch(det, 64, "cuda", fix64=True, log_photons=64 * n)
        mc.mc_simulate_batch(items, W.TINY.n_cdf, src, geo, det, run, t)
        torch.cuda.synchronize()
        out.append([getattr(t, k)[:63].cpu().numpy() for k in ("side", "trans", "scalars")])
    for other in out[1:]:
        for x, y in zip(out[0], other):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("pixels", [1 << 21, 1 << 20, (1 << 20) + 1, 1 << 18, (1 << 18) + 1], ids=str)
@pytest.mark.parametrize("sigma", [False, True], ids=["", "sigma"])
def test_copies_in_the_library_scratch(mc, table, cuda_device, pixels, sigma):
    """One, two, four and eight copies in the library's own scratch: the sums of
    a caller's workspace; a pixel more than it holds is refused."""
    import torch
    n = (1 << 21) + 1 if pixels == 1 << 21 else (1 << 20) + 2
    if sigma:
        pixels = pixels // 2
    w = W.TINY.replace(tau=1.0, n_photons=n, side_px=16, trans_px=16)
    flags = mc.MC_FIX64 | (mc.MC_SIGMA if sigma else 0)
    _, med, src, geo, det, run = mc.args_from_workload(w, table, flags=flags)
    det.side_nx, det.side_ny, det.trans_nx, det.trans_ny = pixels - 48 * 64, 1, 64, 48
    ref, got = (mc.Tally.alloc(det, "cuda", sigma=sigma, fix64=True) for _ in range(2))
    mc.mc_simulate(med, src, geo, det, run, ref)
    mc.mc_simulate_noalloc(med, src, geo, det, run, got)
    torch.cuda.synchronize()
    for k in ("side", "trans", "scalars") + (("side_w2", "trans_w2") if sigma else ()):
        assert torch.equal(getattr(got, k), getattr(ref, k)), k
    if pixels == (1 << 21 if not sigma else 1 << 20):
        det.side_nx += 1
        big = mc.Tally.alloc(det, "cuda", sigma=sigma, fix64=True)
        with pytest.raises(mc.McError):
            mc.mc_simulate_noalloc(med, src, geo, det, run, big)


@pytest.mark.parametrize("sigma", [False, True], ids=["", "sigma"])
@pytest.mark.parametrize("n, shape, overflows", [
    (1 << 21, (1000, 900, 1000, 900), None), ((1 << 21) + 1, (1000, 900, 1000, 900), None),
    (3_000_000, (1024, 1024, 1024, 1024), None), (12_000_000, (1024, 1024, 1024, 1024), True),
    (20_000_000, (1024, 1024, 1024, 1024), None), (5_000_000, (700, 701, 702, 703), None), (9_000_000, (1500, 1200, 64, 48), True),
], ids=str)
def test_a_log_beside_the_copies(mc, table, cuda_device, n, shape, overflows, sigma):
    """Without the flag, a log in the room of unused image copies (not with a grid
    of the caller's): around the counts where it starts and where it no longer
    fits, with and without exits that find it full."""
    import torch
    w = W.TINY.replace(tau=1.0, n_photons=n, side_px=16, trans_px=16)
    out = []
    for blocks in (0, 512):
        _, med, src, geo, det, run = mc.args_from_workload(w, table, flags=mc.MC_FIX64 | (mc.MC_SIGMA if sigma else 0))
        det.side_nx, det.side_ny, det.trans_nx, det.trans_ny = shape
        run.grid_blocks = blocks
        t = mc.Tally.alloc(det, "cuda", sigma=sigma, fix64=True)
        t.workspace.fill_(-1)
        mc.mc_simulate(med, src, geo, det, run, t)
        torch.cuda.synchronize()
        out.append(t)
    full = int(out[0].workspace[21].item())
    if overflows and not sigma:      # (with squares there is twice the room)
        assert full > 0
    for k in ("side", "trans", "scalars") + (("side_w2", "trans_w2") if sigma else ()):
        assert torch.equal(getattr(out[0], k), getattr(out[1], k)), k


@pytest.mark.parametrize("sigma", [False, True], ids=["", "sigma"])
@pytest.mark.parametrize("n_each", [60_000, 400_000])
def test_a_log_beside_the_copies_of_a_batch(mc, table, cuda_device, n_each, sigma):
    import torch
    flags = mc.MC_FIX64 | (mc.MC_SIGMA if sigma else 0)
    _, _, src, geo, det, run = mc.args_from_workload(W.TINY.replace(side_px=150, trans_px=130), table, flags=flags)
    items = [mc.BatchItem(tau=0.1 * (i + 1), albedo=0.9999, inv_cdf=table.inv_cdf.data_ptr(), n_photons=n_each + 77 * i,
                          instance=i) for i in range(40)]
    out = []
    for blocks in (0, 512):
        run.grid_blocks = blocks
        t = mc.Tally.alloc_batch(det, len(items), "cuda", sigma=sigma, fix64=True)
        t.workspace.fill_(-1)
        mc.mc_simulate_batch(items, W.TINY.n_cdf, src, geo, det, run, t)
        torch.cuda.synchronize()
        out.append(t)
    for k in ("side", "trans", "scalars") + (("side_w2", "trans_w2") if sigma else ()):
        assert torch.equal(getattr(out[0], k), getattr(out[1], k)), k

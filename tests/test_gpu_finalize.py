"""From the summed copies to the caller's images (-m gpu): pixel counts at the
edges of a block, images of one pixel, sums written and added, int64 and
double, squared weights in the same launch, the copies of one medium or several.
The oracle walks the same photons; sums of fixed-point weights are exact, so
everything here is compared exactly with them or with each other."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

N = 20_000
SHAPES = [(1, 1, 1, 1), (1, 1023, 32, 32), (1025, 1, 1, 1), (32, 32, 3, 683), (45, 91, 1, 1), (7, 3, 64, 32),
          (64, 64, 4095, 1), (17, 241, 64, 128), (63, 65, 3, 2731), (200, 123, 256, 80)]    # and of 4096


@pytest.fixture(scope="module")
def mc():
    import paper_2507_23189_amd as m
    m.lib()
    return m


@pytest.fixture(scope="module")
def table(mc, cuda_device):
    return mc.mie_table_build(mc.args_from_workload(W.TINY)[0], cuda_device)


def _args(mc, table, shape, flags=0, tau=1.0):
    w = W.TINY.replace(tau=tau, n_photons=N, side_px=16, trans_px=16)
    _, med, src, geo, det, run = mc.args_from_workload(w, table, flags=flags)
    det.side_nx, det.side_ny, det.trans_nx, det.trans_ny = shape
    return med, src, geo, det, run


def _run(mc, args, tally, times=1):
    import torch
    for _ in range(times):
        mc.mc_simulate(*args, tally)
    torch.cuda.synchronize()
    return {k: getattr(tally, k).cpu().numpy().ravel() for k in ("side", "trans", "scalars", "side_w2", "trans_w2")
            if getattr(tally, k, None) is not None}


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("log", [False, True], ids=["atomic", "log"])
def test_images_and_totals_at_the_edges_of_a_block(mc, table, cuda_device, shape, log):
    """int64, double, squared weights and added sums of one walk agree, and the
    faces' totals are those of one-pixel images, which count every exit."""
    extra = mc.MC_EXIT_LOG if log else 0
    fixed = _args(mc, table, shape, mc.MC_FIX64 | extra)
    fixed[4].grid_blocks = 256 if log else 0    # (a launch this small takes the log only if the grid is set)
    got = _run(mc, fixed, mc.Tally.alloc(fixed[3], "cuda", fix64=True, log_photons=N))
    one = _args(mc, table, (1, 1, 1, 1), mc.MC_FIX64)
    ref = _run(mc, one, mc.Tally.alloc(one[3], "cuda", fix64=True))
    assert got["scalars"][mc.MC_S_FACE + 1] == ref["side"][0] / 2.0**32 == got["side"].sum() / 2.0**32
    assert got["scalars"][mc.MC_S_FACE + 5] == ref["trans"][0] / 2.0**32 == got["trans"].sum() / 2.0**32
    assert np.array_equal(got["scalars"], ref["scalars"])

    real = _args(mc, table, shape, mc.MC_SIGMA)
    t = mc.Tally.alloc(real[3], "cuda", sigma=True)
    for img in (t.side, t.trans, t.side_w2, t.trans_w2, t.scalars):
        img.fill_(7.0)                       # written whole, not added to
    dbl = _run(mc, real, t)
    assert np.array_equal(dbl["scalars"], ref["scalars"])
    for k in ("side", "trans"):
        assert np.array_equal(dbl[k], got[k] / 2.0**32), k
        assert 0.0 <= dbl[k + "_w2"].sum() <= dbl[k].sum()

    for flags, base in ((mc.MC_FIX64, got), (0, dbl)):
        acc = _args(mc, table, shape, flags | extra | mc.MC_ACCUMULATE)
        acc[4].grid_blocks = fixed[4].grid_blocks
        t = mc.Tally.alloc(acc[3], "cuda", fix64=bool(flags), log_photons=N)
        for img in (t.side, t.trans, t.scalars):
            img.fill_(3)
        two = _run(mc, acc, t, times=2)
        for k in ("side", "trans", "scalars"):
            assert np.array_equal(two[k], 3 + base[k] + base[k]), k


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_media_of_a_batch_keep_their_own_images(mc, table, cuda_device, shape):
    import torch
    med, src, geo, det, run = _args(mc, table, shape, mc.MC_FIX64)
    taus = (0.25, 1.0, 3.0)
    items = [mc.BatchItem(tau=t, albedo=0.9999, inv_cdf=table.inv_cdf.data_ptr(), n_photons=N, instance=0) for t in taus]
    tally = mc.Tally.alloc_batch(det, len(items), "cuda", fix64=True)
    mc.mc_simulate_batch(items, W.TINY.n_cdf, src, geo, det, run, tally)
    torch.cuda.synchronize()
    for i, tau in enumerate(taus):
        alone = _args(mc, table, shape, mc.MC_FIX64, tau=tau)
        ref = _run(mc, alone, mc.Tally.alloc(det, "cuda", fix64=True))
        for k in ("side", "trans", "scalars"):
            assert np.array_equal(getattr(tally, k)[i].cpu().numpy().ravel(), ref[k]), (tau, k)


@pytest.mark.parametrize("shape", [(64, 64, 100, 100), (200, 123, 256, 80)], ids=str)
def test_pixels_keep_their_places(mc, table, cuda_device, shape):
    """The exits of recorded photons, put into pixels here, give the images."""
    import torch
    med, src, geo, det, run = _args(mc, table, shape, mc.MC_RECORD)
    t = mc.Tally.alloc(det, "cuda", record_rows=N)
    mc.mc_simulate(med, src, geo, det, run, t)
    torch.cuda.synchronize()
    face, (x, y, z), w = t.rec_i[0].cpu().numpy(), t.rec_f[:3].cpu().numpy(), t.rec_f[6].cpu().numpy()
    sx, sy, sz = geo.size_mm

    def index(v, size, n):
        return np.clip((v.astype(np.float32) * np.float32(n / size)).astype(int), 0, n - 1)
    for f, img, row, col in ((1, t.side, index(y, sy, shape[1]), index(z, sz, shape[0])),
                             (5, t.trans, index(y, sy, shape[3]), index(x, sx, shape[2]))):
        ref = np.zeros(img.shape)
        on = face == f
        np.add.at(ref, (row[on], col[on]), w[on])
        # A photon on a pixel's edge may round into the next one.
        moved = np.abs(img.cpu().numpy() - ref).sum()
        assert on.sum() > 100 and moved <= 2e-3 * ref.sum()


@pytest.mark.parametrize("flags", [0, 1], ids=["double", "int64"])
@pytest.mark.parametrize("shape", [(1, 1, 4096, 1), (1, 4095, 64, 65), (200, 123, 256, 80), (181, 181, 5, 3)], ids=str)
def test_copies_in_another_order(mc, table, cuda_device, shape, flags):
    """Past 2^22 photons the copies hold the pixels of each whole block of 4096
    in another order (the exit log does not): written and added images."""
    flags = mc.MC_FIX64 if flags else 0
    out = []
    for extra, times, n in ((mc.MC_EXIT_LOG, 1, (1 << 22) + 1), (0, 1, (1 << 22) + 1),
                            (mc.MC_ACCUMULATE, 2, (1 << 22) + 1), (0, 1, 1 << 22), (mc.MC_EXIT_LOG, 1, 1 << 22)):
        args = _args(mc, table, shape, flags | extra, tau=0.5)
        args[4].n_photons = n
        t = mc.Tally.alloc(args[3], "cuda", fix64=bool(flags), log_photons=n)
        for img in (t.side, t.trans, t.scalars):
            img.fill_(0)
        out.append(_run(mc, args, t, times))
    for k in ("side", "trans", "scalars"):
        assert np.array_equal(out[0][k], out[1][k]) and np.array_equal(2 * out[0][k], out[2][k]), k
        assert np.array_equal(out[3][k], out[4][k]), k


@pytest.mark.parametrize("shape", [(45, 91, 1, 1), (64, 65, 64, 64)], ids=str)
def test_copies_of_a_batch_in_another_order(mc, table, cuda_device, shape):
    import torch
    med, src, geo, det, run = _args(mc, table, shape, mc.MC_FIX64)
    out = []
    for flags in (mc.MC_FIX64, mc.MC_FIX64 | mc.MC_EXIT_LOG):
        det.flags = flags
        items = [mc.BatchItem(tau=0.3 * (i + 1), albedo=0.9999, inv_cdf=table.inv_cdf.data_ptr(), n_photons=2_000_000,
                              instance=i) for i in range(3)]
        t = mc.Tally.alloc_batch(det, 3, "cuda", fix64=True, log_photons=6_000_000)
        mc.mc_simulate_batch(items, W.TINY.n_cdf, src, geo, det, run, t)
        torch.cuda.synchronize()
        out.append(t)
    for k in ("side", "trans", "scalars"):
        assert torch.equal(getattr(out[0], k), getattr(out[1], k)), k

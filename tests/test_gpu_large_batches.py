"""The largest batches (-m gpu), whose tallies fill half a CU's LDS to the byte: the
block's pool of work units and its count of exits past the log share the first
medium's tally words, so that medium's totals are looked at as well."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("media, log", [(512, False), (512, True), (384, True), (1, False), (1, True)], ids=str)
def test_media_of_the_largest_batches(cuda_device, media, log):
    import torch
    import paper_2507_23189_amd as mc
    table = mc.mie_table_build(mc.args_from_workload(W.TINY)[0], cuda_device)
    flags = mc.MC_FIX64 | (mc.MC_EXIT_LOG if log else 0)
    n = max(4000, 2_200_000 // media)        # with the flag, past the count from which the log is used
    _, med, src, geo, det, run = mc.args_from_workload(W.TINY.replace(side_px=16, trans_px=16), table, flags=flags)
    items = [mc.BatchItem(tau=0.25 + 0.5 * (i % 7), albedo=0.999, inv_cdf=table.inv_cdf.data_ptr(), n_photons=n + i,
                          instance=i) for i in range(media)]
    # A log with hardly any room: the count of the exits that found it full.
    t = mc.Tally.alloc_batch(det, media, "cuda", fix64=True, log_photons=media * n // 8)
    mc.mc_simulate_batch(items, W.TINY.n_cdf, src, geo, det, run, t)
    torch.cuda.synchronize()
    s = t.scalars.cpu().numpy()
    assert np.array_equal(s[:, mc.MC_S_PHOTONS], n + np.arange(media))
    for k, img in ((1, t.side), (5, t.trans)):
        assert np.array_equal(s[:, k], img.sum(dim=(1, 2)).double().cpu().numpy() * 2.0**-32)
    run.n_photons, run.instance = n, 0
    for i in sorted({0, 1 % media, media - 1}):
        med.tau, med.albedo = items[i].tau, items[i].albedo
        run.n_photons, run.instance = n + i, i
        det.flags = mc.MC_FIX64
        one = mc.Tally.alloc(det, "cuda", fix64=True)
        mc.mc_simulate(med, src, geo, det, run, one)
        torch.cuda.synchronize()
        assert np.array_equal(one.scalars.cpu().numpy()[:15], s[i][:15])
        assert torch.equal(one.side, t.side[i]) and torch.equal(one.trans, t.trans[i])

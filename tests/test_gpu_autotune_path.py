"""The batch tuner times the tally path that the whole launch takes (-m gpu)."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flag", [True, False], ids=["flag", "beside the copies"])
def test_a_sample_goes_through_the_log_of_its_launch(cuda_device, flag):
    """64 media of 40,000 photons go through the exit log; a sixteenth of them alone
    would not.  The log's counts, which every walk with it writes, show it."""
    import torch
    import paper_2507_23189_amd as mc
    table = mc.mie_table_build(mc.args_from_workload(W.TINY)[0], cuda_device)
    w = W.TINY.replace(side_px=96, trans_px=96)
    _, _, src, geo, det, run = mc.args_from_workload(w, table, flags=mc.MC_FIX64 | (mc.MC_EXIT_LOG if flag else 0))
    items = [mc.BatchItem(tau=0.5 + 0.1 * i, albedo=0.999, inv_cdf=table.inv_cdf.data_ptr(), n_photons=40_000, instance=i)
             for i in range(64)]
    t = mc.Tally.alloc_batch(det, 64, "cuda", fix64=True, log_photons=64 * 40_000)
    # The counts follow the workspace and the schedule, or the copies in use: two, with
    # which 2^8 ranges of keys make 512 blocks of the binning kernel.
    pixels = 64 * 2 * 96 * 96
    at = mc.mc_workspace_bytes_batch(mc.Detector(96, 96, 96, 96, mc.MC_FIX64), 64) // 8 if flag else 64 * 32 + 2 * pixels
    seen = []
    for call in ("simulate", "tune"):
        t.workspace.fill_(-1)
        if call == "simulate":
            mc.mc_simulate_batch(items, W.TINY.n_cdf, src, geo, det, run, t)
        else:
            mc.mc_autotune_batch(items, W.TINY.n_cdf, src, geo, det, run, t, 1.0 / 16)
        torch.cuda.synchronize()
        counts = t.workspace[at:at + 4096].view(torch.int32)
        seen.append(int(counts.min()) >= 0 and int(counts.max()) > 0)
    assert seen == [True, True]

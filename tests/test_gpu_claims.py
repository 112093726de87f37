"""How photon ids reach the lanes (-m gpu): shares dealt out, pools refilled from
the counter, launches with more blocks than ids, chunks of one id and larger
than the launch.  Every id is walked once whatever the shape: fixed-point
images and scalars equal those of one block and of the standalone runs."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

N = 70_001
NAMES = ("side", "trans", "scalars")


@pytest.fixture(scope="module")
def mc():
    import paper_2507_23189_amd as m
    m.lib()
    return m


@pytest.fixture(scope="module")
def table(mc, cuda_device):
    return mc.mie_table_build(mc.args_from_workload(W.TINY)[0], cuda_device)


def _run(mc, table, n=N, tau=2.0, **shape):
    import torch
    w = W.TINY.replace(tau=tau, n_photons=n, side_px=16, trans_px=16)
    _, med, src, geo, det, run = mc.args_from_workload(w, table, flags=mc.MC_FIX64)
    for k, v in shape.items():
        setattr(run, k, v)
    t = mc.Tally.alloc(det, "cuda", fix64=True)
    mc.mc_simulate(med, src, geo, det, run, t)
    torch.cuda.synchronize()
    return {k: getattr(t, k).cpu().numpy() for k in NAMES}


@pytest.mark.parametrize("shape", [
    dict(),                                             # shares of a full launch
    dict(grid_blocks=1),                                # one block that refills its pool
    dict(grid_blocks=3, chunk=1), dict(grid_blocks=3, chunk=65536), dict(grid_blocks=16, chunk=37),
    dict(grid_blocks=5, block_size=64), dict(grid_blocks=4000, block_size=64), dict(grid_blocks=1000, chunk=100),
], ids=str)
def test_every_id_is_walked_once(mc, table, cuda_device, shape):
    ref = _run(mc, table, grid_blocks=2, block_size=1024, chunk=64)
    got = _run(mc, table, **shape)
    assert got["scalars"][mc.MC_S_PHOTONS] == N
    for k in NAMES:
        assert np.array_equal(got[k], ref[k]), k


@pytest.mark.parametrize("n", [1, 64, 2_097_152, 2_097_153, 5_000_000])   # to four photons per lane, and past it
def test_photons_counted_at_the_edges_of_the_shares(mc, table, cuda_device, n):
    got = _run(mc, table, n=n, tau=0.5)
    assert got["scalars"][mc.MC_S_PHOTONS] == n


@pytest.mark.parametrize("shape", [dict(), dict(chunk=1), dict(chunk=64, grid_blocks=2), dict(grid_blocks=3000)], ids=str)
def test_batch_units_are_walked_once(mc, cuda_device, shape):
    import torch
    counts = [1, 0, 5000, 64, 20_011, 3]
    tau = [0.5, 1.0, 4.0, 2.0, 1.0, 3.0]
    table = mc.mie_table_build(mc.args_from_workload(W.TINY)[0], cuda_device)
    _, _, src, geo, det, run = mc.args_from_workload(W.TINY.replace(side_px=16, trans_px=16), table, flags=mc.MC_FIX64)
    for k, v in shape.items():
        setattr(run, k, v)
    items = [mc.BatchItem(tau=t, albedo=0.9999, inv_cdf=table.inv_cdf.data_ptr(), n_photons=n, instance=0)
             for t, n in zip(tau, counts)]
    tb = mc.Tally.alloc_batch(det, len(items), "cuda", fix64=True)
    mc.mc_simulate_batch(items, W.TINY.n_cdf, src, geo, det, run, tb)
    torch.cuda.synchronize()
    for i, (t, n) in enumerate(zip(tau, counts)):
        one = _run(mc, table, n=n, tau=t)
        for k in NAMES:
            assert np.array_equal(getattr(tb, k)[i].cpu().numpy(), one[k]), (i, k)


@pytest.mark.parametrize("tau, per_lane", [(0.5, 3), (4.0, 4), (8.0, 5), (16.0, 0.5), (16.0, 5)], ids=str)
@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_one_block_per_cu_or_two(mc, table, cuda_device, tau, per_lane, extra):
    """Around the photon counts where a launch takes two blocks per CU instead
    of one (or one instead of two): the sums of a fixed grid."""
    import torch
    lanes = torch.cuda.get_device_properties(0).multi_processor_count * 1024
    n = int(per_lane * lanes) + extra
    got, ref = _run(mc, table, n=n, tau=tau), _run(mc, table, n=n, tau=tau, grid_blocks=300)
    for k in NAMES:
        assert np.array_equal(got[k], ref[k]), k

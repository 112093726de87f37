"""The log that walks without the flag keep among unused image copies (-m gpu), in the
forms a walk has: HG, a finite beam, path moments, accumulation, double images, the
library's own scratch.  A grid of the caller's takes the atomics."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

SHAPE, N = (1000, 900, 1000, 900), 3_000_000


@pytest.fixture(scope="module")
def mc():
    import paper_2507_23189_amd as m
    m.lib()
    return m


@pytest.fixture(scope="module")
def table(mc, cuda_device):
    return mc.mie_table_build(mc.args_from_workload(W.TINY)[0], cuda_device)


def _walk(mc, table, grid, flags, *, shape=SHAPE, times=1, noalloc=False, moments=False, **kw):
    """The tally, and whether the walk kept a log in place of its last image copy."""
    import torch
    from paper_2507_23189_amd import _capi as K
    flags |= K.MC_MOMENTS if moments else 0
    w = W.TINY.replace(tau=2.0, n_photons=N, side_px=16, trans_px=16, **kw)
    _, med, src, geo, det, run = mc.args_from_workload(w, table, flags=flags, grid_blocks=grid)
    det.side_nx, det.side_ny, det.trans_nx, det.trans_ny = shape
    t = mc.Tally.alloc(det, "cuda", fix64=bool(flags & mc.MC_FIX64), moments=moments)
    for img in (t.side, t.trans, t.scalars, t.side_wk, t.side_wl):
        if img is not None:
            img.zero_()
    t.workspace.fill_(-1)
    for i in range(times):
        run.photon_offset = i * N
        (mc.mc_simulate_noalloc if noalloc else mc.mc_simulate)(med, src, geo, det, run, t)
    torch.cuda.synchronize()
    # With atomics all eight copies are cleared; the log leaves some of its places as
    # they were.
    pixels = shape[0] * shape[1] + shape[2] * shape[3]
    return t, bool((t.workspace[32 + 7 * pixels:32 + 8 * pixels] == -1).any())


@pytest.mark.parametrize("form", ["mie", "hg", "beam", "moments", "accumulate", "double", "roulette"])
def test_forms_of_a_walk(mc, table, cuda_device, form):
    import torch
    kw = dict(hg=dict(phase=W.PHASE_HG), beam=dict(beam_radius_mm=1.25), moments=dict(moments=True), accumulate=dict(times=2),
              roulette=dict(roulette_w=0.5, roulette_p=0.2, albedo=0.9)).get(form, {})
    flags = (0 if form == "double" else mc.MC_FIX64) | (mc.MC_ACCUMULATE if form == "accumulate" else 0)
    a, log = _walk(mc, table, 0, flags, **kw)
    b, atomics = _walk(mc, table, 512, flags, **kw)
    assert log and not atomics
    for k in ("side", "trans"):
        assert torch.equal(getattr(a, k), getattr(b, k)), k
    assert torch.equal(a.scalars[:15], b.scalars[:15])
    assert float(a.scalars[mc.MC_S_PHOTONS]) == N * kw.get("times", 1)
    if form == "moments":
        # FP64 sums of the same terms in another order: each pixel's and the image's off
        # by at most their number of terms times 2^-53.
        for k in ("side_wk", "side_wl"):
            np.testing.assert_allclose(getattr(a, k).cpu().numpy(), getattr(b, k).cpu().numpy(), rtol=N * 2.0**-53)
        np.testing.assert_allclose(a.scalars[16:19].cpu().numpy(), b.scalars[16:19].cpu().numpy(), rtol=N * 2.0**-53)


def test_in_the_library_scratch(mc, table, cuda_device):
    """Four copies of these images fill its 2^21 words and leave no room for a log: the
    same sums."""
    import torch
    shape = (500, 512, 500, 512)
    a, _ = _walk(mc, table, 0, mc.MC_FIX64, shape=shape, noalloc=True)   # (its workspace is not looked at)
    b, _ = _walk(mc, table, 512, mc.MC_FIX64, shape=shape, noalloc=True)
    c, _ = _walk(mc, table, 512, mc.MC_FIX64, shape=shape)
    for other in (b, c):
        assert torch.equal(a.side, other.side) and torch.equal(a.trans, other.trans)
        assert torch.equal(a.scalars[:15], other.scalars[:15])

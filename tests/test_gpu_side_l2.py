"""The L2 loss of a side image and its derivative in one pass (-m gpu), at the
edges of a block's 2048 pixels, in a workspace with room for few blocks, and
beside targets that the pass does not take.

A sum of n squares in any order and with fused products is off by at most
n 2^-53 of itself, and so is the reference's; the derivative is exact."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (1, 2047), (2, 1024), (683, 3), (64, 64), (300, 257), (1024, 1030)]


@pytest.fixture(scope="module")
def mc():
    import paper_2507_23189_amd as m
    m.lib()
    return m


def _tally(mc, shape, dev):
    import torch
    rng = torch.Generator().manual_seed(shape[0] * 4099 + shape[1])
    det = mc.Detector(shape[1], shape[0], 1, 1, mc.MC_MOMENTS)
    t = mc.Tally.alloc(det, dev, moments=True)
    for img in (t.side, t.side_wk, t.side_wl):
        img.copy_(torch.rand(shape, generator=rng, dtype=torch.float64) * 1e3)
    t.scalars.copy_(torch.rand(mc.MC_N_SCALARS, generator=rng, dtype=torch.float64))
    return det, t, (torch.rand(shape, generator=rng, dtype=torch.float64) * 1e3).to(dev)


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("words", [0, 33, 35])
def test_loss_and_derivative(mc, cuda_device, shape, words):
    import torch
    det, t, target = _tally(mc, shape, cuda_device)
    if words:                    # as few partials as the smallest workspaces hold
        det_ws = torch.empty(words, dtype=torch.int64, device=cuda_device)
        t.workspace = det_ws
        tc = t._c()
        g, loss = torch.empty_like(t.side), torch.empty((), dtype=torch.float64, device=cuda_device)
        rc = mc.lib().mc_side_l2(det, tc, target.data_ptr(), g.data_ptr(), loss.data_ptr(), None)
        assert rc == 0
        torch.cuda.synchronize()
    else:
        loss, g = mc.mc_side_l2(det, t, target)
    diff = t.side.cpu() - target.cpu()
    assert torch.equal(g.cpu(), 2.0 * diff)
    ref = (diff * diff).numpy().astype(np.longdouble).sum()
    w2 = float(t.scalars[mc.MC_S_SIDE_W2])
    assert abs(np.longdouble(float(loss)) - (ref - w2)) <= (diff.numel() + 2) * 2.0**-53 * ref + 2.0**-52 * w2


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("pixel2", [False, True])
def test_dot_products_of_the_gradient(mc, cuda_device, shape, pixel2):
    import torch
    det, t, g = _tally(mc, shape, cuda_device)
    med = mc.Medium(input=mc.MC_MEDIUM_MU, phase=mc.MC_PHASE_HG, g=0.9, mu_sca=0.5, mu_abs=0.0)
    geo = mc.Geometry()
    for i in range(3):
        geo.size_mm[i] = 10.0
    geo.n_medium = geo.n_outside = 1.0
    h = None
    if pixel2:
        h = g.flip(0).contiguous()
        t.side_w2k, t.side_w2l = t.side_wl.clone(), t.side_wk.clone()
    got = mc.mc_grad(med, geo, det, t, g, h)
    f = [x.cpu().numpy().astype(np.longdouble) for x in (g, t.side_wk, t.side_wl)]
    k, l = (f[0] * f[1]).sum(), (f[0] * f[2]).sum()
    qk = ql = np.longdouble(0)
    if pixel2:
        fh = h.cpu().numpy().astype(np.longdouble)
        qk, ql = (fh * f[2]).sum(), (fh * f[1]).sum()
    # All terms are positive: each dot is off by at most n 2^-53 of itself, the
    # few operations after it by 2^-53 of what they join.
    size = k / 0.5 + l + qk / 0.5 + ql
    tol = (g.numel() + 8) * 2.0**-53 * size
    assert abs(got[0] - float((k / 0.5 - l) - (qk / 0.5 - ql))) <= tol
    assert abs(got[1] - float(-l + ql)) <= tol


@pytest.mark.parametrize("kind", ["image", "float32", "row", "strided", "scalar"])
def test_targets_of_any_form(mc, cuda_device, kind):
    """side_l2_loss takes what the tensor expression takes."""
    import torch
    table = mc.mie_table_build(mc.args_from_workload(W.TINY)[0], cuda_device)
    w = W.TINY.replace(tau=2.0, n_photons=20_000, side_px=40, trans_px=8)
    _, med, src, geo, det, run = mc.args_from_workload(w, table)
    walks = []

    class Kept(mc.SideImage):        # the moments' atomics add in another order in another walk
        def run_walk(self, *mu):
            walks.append(super().run_walk(*mu))
            return walks[-1]
    sim = Kept(med, src, geo, det, run)
    target = torch.rand((40, 40), dtype=torch.float64, device=cuda_device)
    target = {"image": target, "float32": target.float(), "row": target[3], "strided": target.t(),
              "scalar": torch.tensor(0.25, dtype=torch.float64, device=cuda_device)}[kind]
    mu = [torch.tensor(v, dtype=torch.float64, requires_grad=True) for v in (0.2, 1e-4)]
    loss = mc.side_l2_loss(mu[0], mu[1], target, sim)
    loss.backward()
    (_, t), = walks
    diff = t.side - target
    sq = float((diff * diff).sum())
    w2 = float(t.scalars[mc.MC_S_SIDE_W2])
    tol = 2 * 1600 * 2.0**-53
    assert abs(float(loss.detach()) - (sq - w2)) <= tol * (sq + w2)
    ref = mc.mc_grad(sim.medium_for(0.2, 1e-4), geo, sim.detector, t, (2.0 * diff).contiguous(), d2loss_uniform=2.0)
    assert [m.grad.item() for m in mu] == pytest.approx(list(ref[:2]), rel=1e-12)


def test_refusals(mc, cuda_device):
    import torch
    det, t, target = _tally(mc, (4, 4), cuda_device)
    with pytest.raises(ValueError):
        mc.mc_side_l2(det, t, target.float())
    with pytest.raises(ValueError):
        mc.mc_side_l2(det, t, target[:3])
    with pytest.raises(ValueError):
        mc.mc_side_l2(det, t, target.cpu())
    t.workspace = torch.empty(32, dtype=torch.int64, device=cuda_device)
    tc = t._c()
    g = torch.empty_like(t.side)
    assert mc.lib().mc_side_l2(det, tc, target.data_ptr(), g.data_ptr(), g.data_ptr(), None) == mc.MC_EINVAL
    assert mc.lib().mc_side_l2(det, tc, None, g.data_ptr(), g.data_ptr(), None) == mc.MC_EINVAL

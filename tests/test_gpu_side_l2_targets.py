"""The L2 loss against targets whose memory does not hold their values (-m gpu)."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["negated", "zero"])
def test_views_without_values_in_memory(cuda_device, kind):
    import torch
    import paper_2507_23189_amd as mc
    table = mc.mie_table_build(mc.args_from_workload(W.TINY)[0], cuda_device)
    w = W.TINY.replace(tau=2.0, n_photons=20_000, side_px=40, trans_px=8)
    sim = mc.SideImage(*mc.args_from_workload(w, table)[1:])
    values = torch.rand((40, 40), dtype=torch.float64, device=cuda_device)
    target = torch._neg_view(values) if kind == "negated" else torch._efficientzerotensor(
        (40, 40), dtype=torch.float64, device=cuda_device)
    plain = -values if kind == "negated" else torch.zeros_like(values)
    out = []
    for t in (target, plain):
        mu = [torch.tensor(v, dtype=torch.float64, requires_grad=True) for v in (0.2, 1e-4)]
        loss = mc.side_l2_loss(mu[0], mu[1], t, sim)
        loss.backward()
        out.append([float(loss.detach())] + [m.grad.item() for m in mu])
    # The same photons: the image's sums are exact, the moments' FP64 sums of up to
    # 2e4 terms are in another order in each walk.
    assert out[0] == pytest.approx(out[1], rel=1e-9)

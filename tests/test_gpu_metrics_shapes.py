"""The image measures at the edges of their tiles and blocks (-m gpu): one pixel,
one column, one row, widths around a tile's 64 columns, heights around its 64
rows, more pixels than the blocks take at once, one annulus and the most."""
import numpy as np
import pytest

from oracle import metrics as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,r_max", [
    (1, 1, 0.9), (1, 300, 40.0), (300, 1, 40.0), (2, 1025, 2.0), (63, 15, 7.5), (64, 16, 8.0), (65, 17, 30.0),
    (64, 63, 1.0), (127, 129, 64.0), (64, 65, 20.0), (31, 2000, 1000.0), (1030, 1031, 515.5), (2050, 100, 2048.0)])
@pytest.mark.parametrize("third", [False, True])
def test_measures_match_the_oracle(cuda_device, nx, ny, r_max, third):
    import torch
    import paper_2507_23189_amd as mc
    rng = np.random.default_rng([nx, ny])
    a, b, c = rng.random((3, ny, nx)) + 0.01
    cx, cy = 0.5 * nx + 0.25, 0.5 * ny
    dev = [torch.tensor(v, device=cuda_device) for v in (a, b, c)]
    g = mc.image_metrics(dev[0], dev[1], dev[2] if third else None, cx=cx, cy=cy, r_max=r_max, profiles=True)
    o = M.image_metrics(a, b, cx, cy, r_max, c=c if third else None)
    assert g["max"][:2] == [a.max(), b.max()] and g["pixels"] == nx * ny
    np.testing.assert_array_equal(g["count"].cpu().numpy(), o["count"])
    # Annulus means of values up to 1 held to 2^-39 each; FP64 sums elsewhere.
    for k in ("profile_a", "profile_b"):
        np.testing.assert_allclose(g[k].cpu().numpy(), o[k], rtol=0, atol=4e-12)
    for k in ("rmse", "r", "radial_r"):
        if np.isnan(o[k]) or (k != "rmse" and min(nx * ny, (o["count"] > 0).sum()) < 3):
            continue   # no spread to correlate
        assert abs(g[k] - o[k]) <= 1e-9, k
    np.testing.assert_allclose(g["zone_rmse"], o["zone_rmse"], rtol=0, atol=1e-10)
    again = mc.image_metrics(dev[0], dev[1], dev[2] if third else None, cx=cx, cy=cy, r_max=r_max)
    assert all(again[k] == g[k] or again[k] != again[k] for k in ("rmse", "r", "radial_r", "zone_rmse"))

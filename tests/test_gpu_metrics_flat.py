"""The image measures of flat images (-m gpu), whose tiles have fewer rows and more
columns: at the edges of both."""
import numpy as np
import pytest

from oracle import metrics as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [
    (65, 1), (4095, 1), (4096, 1), (4097, 1), (40_000, 1), (2049, 2), (5000, 2), (1500, 3), (1025, 4), (4100, 4), (513, 5),
    (1030, 8), (600, 9), (257, 16), (300, 17), (1000, 31), (129, 32), (700, 33), (63, 33), (64, 20), (70_000, 20)], ids=str)
@pytest.mark.parametrize("third", [False, True])
def test_flat_images_match_the_oracle(cuda_device, nx, ny, third):
    import torch
    import paper_2507_23189_amd as mc
    rng = np.random.default_rng([nx, ny])
    a, b, c = rng.random((3, ny, nx)) + 0.01
    cx, cy, r_max = 0.5 * nx + 0.25, 0.5 * ny, min(0.4 * nx, 2000.0)
    dev = [torch.tensor(v, device=cuda_device) for v in (a, b, c)]
    g = mc.image_metrics(dev[0], dev[1], dev[2] if third else None, cx=cx, cy=cy, r_max=r_max, profiles=True)
    o = M.image_metrics(a, b, cx, cy, r_max, c=c if third else None)
    assert g["max"][:2] == [a.max(), b.max()] and g["pixels"] == nx * ny
    np.testing.assert_array_equal(g["count"].cpu().numpy(), o["count"])
    # Annulus means of values up to 1 held to 2^-39 each; FP64 sums elsewhere.
    for k in ("profile_a", "profile_b"):
        np.testing.assert_allclose(g[k].cpu().numpy(), o[k], rtol=0, atol=4e-12)
    for k in ("rmse", "r", "radial_r"):
        assert abs(g[k] - o[k]) <= 1e-9, k
    np.testing.assert_allclose(g["zone_rmse"], o["zone_rmse"], rtol=0, atol=1e-10)

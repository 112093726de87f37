"""The table's recurrences and sums at the edges of their chunks and groups
(-m gpu): series of one to a few terms, term counts around the groups of eight
terms, starts around the chunks of 256 steps, a real and an absorbing index
(whose downward steps differ), an index so large that |m| x sets the start, and
angle counts around a workgroup's 64."""
import numpy as np
import pytest

from oracle import mie

pytestmark = pytest.mark.gpu

N_MED, LAMBDA = 1.33, 532.0


def _diameter(x):
    return x * LAMBDA / (np.pi * 1e3 * N_MED)


@pytest.mark.parametrize("m_im", [0.0, 0.02])
@pytest.mark.parametrize("x,m_re,n_angles", [
    (1e-3, 1.59, 3), (0.5, 1.59, 63), (1.0, 1.59, 64), (2.0, 1.59, 65), (6.0, 1.59, 128), (7.3, 1.59, 129), (9.5, 1.2, 257),
    (57.0, 1.59, 181), (58.1, 1.59, 181), (146.0, 1.59, 181), (190.0, 1.59, 256), (440.0, 1.59, 181), (12.0, 60.0, 181),
    (30.0, 13.3, 181)])
def test_tables_match_the_oracle(cuda_device, x, m_re, n_angles, m_im):
    import paper_2507_23189_amd as mc
    d = float(_diameter(x))
    spec = mc.MieSpec(n_medium=N_MED, m_re=m_re, m_im=m_im, diameter_um=d, wavelength_nm=LAMBDA, n_angles=n_angles,
                      n_cdf=1000)
    t = mc.mie_table_build(spec, cuda_device, phase=True, cdf=True, coef=True)
    o = mie.build_table(d, m_re, m_im, N_MED, LAMBDA, n_angles, 1000)
    c = t.coef.cpu().numpy()
    scale = max(np.abs(o.a).max(), np.abs(o.b).max())
    # Both sides round the recurrences in FP64: errors grow with the steps taken
    # (1e-15 each, over |m| x steps) and, near resonances of a large real index,
    # with how fast D_n turns (up to |m| times).  Below x = 1 the upward start
    # psi_1 = sin(x) / x - cos(x) cancels down to x^2 / 3, so its few roundings
    # weigh 3 / x^2 times as much, on either side.
    tol = 2e-14 * max(1.0, x * abs(complex(m_re, m_im)) / N_MED) * max(1.0, m_re / N_MED) + 4.0 * 2.2e-16 * 3.0 / x**2
    assert np.abs(c[:, 0] + 1j * c[:, 1] - o.a).max() <= tol * scale
    assert np.abs(c[:, 2] + 1j * c[:, 3] - o.b).max() <= tol * scale
    assert abs(t.q_ext - o.q_ext) <= 10 * tol * o.q_ext and abs(t.q_sca - o.q_sca) <= 10 * tol * o.q_ext
    P = t.phase.cpu().numpy()
    assert np.abs(P - o.P).max() <= 1e2 * tol * o.P.max()
    assert np.abs(t.cdf.cpu().numpy() - o.F).max() <= 1e2 * tol


@pytest.mark.parametrize("m_im", [0.0, 0.001, 0.02])
@pytest.mark.parametrize("x, m_re", [(153.0, 1.59), (195.0, 1.59), (196.0, 1.59), (197.0, 1.59), (232.0, 1.59), (255.0, 1.35),
                                     (268.0, 1.59), (520.0, 1.4), (700.0, 1.59), (850.0, 1.4), (20.0, 17.0), (20.1, 18.0)])
def test_shared_downward_steps(cuda_device, x, m_re, m_im):
    """From 256 downward steps all lanes of a wave share them: starts around that
    and around multiples of 64, and |m| x above the number of terms."""
    test_tables_match_the_oracle(cuda_device, x, m_re, 181, m_im)

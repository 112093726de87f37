"""Strongly absorbing spheres (-m gpu), whose downward steps, from 256 on, are shared
by a wave: the matrices' products then grow by the absorption as well."""
import pytest

from test_gpu_table_steps import test_tables_match_the_oracle as matches_the_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m_im", [0.1, 0.5, 1.33, 6.0])
@pytest.mark.parametrize("x, m_re", [(20.0, 17.0), (150.0, 1.59), (200.0, 1.34), (200.0, 0.2), (440.0, 1.59), (700.0, 1.4)])
def test_shared_steps_of_absorbing_spheres(cuda_device, x, m_re, m_im):
    matches_the_oracle(cuda_device, x, m_re, 181, m_im)

"""Calls that wait for scalar results (-m gpu), on many threads and streams at a
time: every caller gets its own results, the ones a device buffer holds."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_many_threads_get_their_own_results(cuda_device):
    import torch
    import paper_2507_23189_amd as mc
    d = 0.5 + 0.05 * np.arange(16)
    a = [torch.rand(40, 50, dtype=torch.float64, device=cuda_device) for _ in d]

    def work(i):
        spec = mc.MieSpec(n_medium=1.33, m_re=1.59, m_im=0.0, diameter_um=float(d[i]), wavelength_nm=532.0, n_angles=181,
                          n_cdf=64)
        with torch.cuda.stream(torch.cuda.Stream()):
            t = mc.mie_table_build(spec, cuda_device)
            p = mc.mie_table_build_poly(spec, 0.03, 5, cuda_device)
            m = mc.image_metrics(a[i], a[0])
        return t.q_ext, t.g, t.n_terms, p.q_sca, p.n_terms, m["rmse"], m["max"][0]

    torch.cuda.synchronize()
    alone = [work(i) for i in range(len(d))]
    with ThreadPoolExecutor(12) as pool:
        for _ in range(4):
            assert list(pool.map(work, range(len(d)))) == alone


def test_enqueued_builds_leave_the_same_results_on_the_device(cuda_device):
    import torch
    import paper_2507_23189_amd as mc
    spec = mc.MieSpec(n_medium=1.33, m_re=1.59, m_im=0.01, diameter_um=3.0, wavelength_nm=532.0, n_angles=181, n_cdf=64)
    t, e = mc.mie_table_build(spec, cuda_device), mc.mie_table_enqueue(spec, cuda_device)
    torch.cuda.synchronize()
    assert e.result.tolist() == [t.q_ext, t.q_sca, t.g, float(t.n_terms)]

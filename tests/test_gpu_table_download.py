"""dp_table_download takes no host memory beside the caller's array: the peak of
a process that downloads a table of 650 MB grows by that array, not by twice as
much, and the coefficients are the intervals' own quintics (value at the left
node and continuity at the right one, as every interval matches the net at both:
1e-11 of the table's largest value in FP64)."""
import resource

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_no_copy_on_the_host(cu_cfg, cu_params):
    import paper_2201_01446_amd as P
    m = P.Model(cu_cfg, cu_params).tabulate(0.7, 7e-6, 1.4, 1e-4)
    torch.cuda.synchronize()
    peak = lambda: resource.getrusage(resource.RUSAGE_SELF).ru_maxrss * 1024
    P.Model(cu_cfg, cu_params).tabulate(0.7, 0.01, 1.4, 0.1).table()   # what a first copy allocates
    before = peak()
    tab = m.table()
    assert tab.nbytes > 600e6
    assert peak() - before <= 1.5 * tab.nbytes
    n = 100000   # the fine intervals
    assert len(tab) == n + 7000
    k = np.random.default_rng(1).integers(0, n - 1, 200)
    w = 7e-6 ** np.arange(6)
    right, left = (tab[k] * w).sum(-1), tab[k + 1, :, 0]
    assert np.max(np.abs(right - left)) <= 1e-11 * np.max(np.abs(left))

"""Host time of an operator apply: the depth of its blocks is looked up once per mesh, so a
call on a column of 30,000 cells costs the host what one on 50 cells does (the rule of the
Q2 strips goes through all depths of the mesh).  The least of 60 calls, each on an idle GPU;
the factor of 3 is for what the two calls do not share."""
import time

import numpy as np
import pytest

from gpu_util import print_case

pytestmark = pytest.mark.gpu


def _host_time(hts, nz):
    import torch
    n = (2, 2, nz)
    m = hts.Mesh((0.0, 0.0, 0.0), (10.0, 10.0, float(nz)), n, 2)
    one = np.ones(m.ncell)
    m.set_materials(1e-12 * one, 0.3 * one, 2.5 * one, 2e6 * one, 1000.0, 1e-3, 4.18e6, 0.6, 9.81, 1e5)
    x = torch.ones(m.nnode, dtype=torch.float64, device="cuda:0")
    y = torch.zeros_like(x)
    best = 1e9
    for _ in range(60):
        torch.cuda.synchronize()
        t = time.perf_counter()
        m.apply_operator(0, 0, 86400.0, x, y)
        best = min(best, time.perf_counter() - t)
    torch.cuda.synchronize()
    return best


def test_host_time_does_not_grow_with_the_height(hts):
    print_case("host time of an apply")
    low, high = _host_time(hts, 50), _host_time(hts, 30000)
    print("us: %.1f %.1f" % (1e6 * low, 1e6 * high))
    assert high <= 3.0 * low

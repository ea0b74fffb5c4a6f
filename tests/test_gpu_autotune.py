"""The autotuner's candidate depths: they rise, none is left out, and the search ends before
the deepest one only past two depths in a row at which both precisions take more than 1.6
times their best (from the lines it prints with HTS_VERBOSE, in a process of its own because
the variable is read once)."""
import os
import re
import subprocess
import sys

import pytest

from gpu_util import print_case

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RUN = """
import numpy as np
import paper_2103_00081_amd as hts
import synth
n, degree, hexa = {n}, {degree}, {hexa}
ext = (1000.0, 1000.0, 200.0)
m = hts.Mesh((0.0, 0.0, 0.0), ext, n, degree, coords=synth.terrain_coords((0.0, 0.0, 0.0), ext, n) if hexa else None)
one = np.ones(m.ncell)
m.set_materials(1e-12 * one, 0.3 * one, 2.5 * one, 2e6 * one, 1000.0, 1e-3, 4.18e6, 0.6, 9.81, 1e5)
hts.autotune([m])
"""
USUAL = [2, 3, 4, 5, 6, 8, 10, 12, 16, 24, 32, 48, 64]


@pytest.mark.parametrize("n,degree,hexa", [((96, 96, 48), 2, False), ((7, 5, 2), 2, False), ((96, 80, 40), 1, True),
                                           ((64, 64, 32), 1, False)],
                         ids=["q2", "q2 5 planes", "hexahedra", "q1"])
def test_all_depths_are_timed(n, degree, hexa):
    print_case("autotune", n, degree, hexa)
    env = dict(os.environ, HTS_VERBOSE="1")
    env.pop("HTS_TUNE_CACHE", None)
    r = subprocess.run([sys.executable, "-c", RUN.format(n=n, degree=degree, hexa=hexa)], cwd=ROOT, env=env,
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=110)
    assert r.returncode == 0, r.stdout[-2000:]
    runs = {}
    for fam, field, z, a, b in re.findall(r"autotune family (\d+) field (\d) \S+ z-depth (\d+): (\S+) us FP64, (\S+) us FP32",
                                          r.stdout):
        runs.setdefault((int(fam), int(field)), []).append((int(z), float(a), float(b)))
    assert len(runs) == 4                                   # two kernel families, two fields
    planes = degree * n[2] + 1
    whole = lambda z: (min(z, planes) + 1) // 2 * 2 if degree == 2 else min(z, planes)
    for key, t in runs.items():
        depths = [z for z, _, _ in t]
        assert depths == sorted(depths), (key, depths)
        done = [whole(z) for z in depths]
        assert len(set(done)) == len(done)
        full = [z for z in USUAL if z <= planes]
        last = depths[-1]
        for z in full:
            assert z > last or whole(z) in done, (key, z, depths)
        if last < full[-1] and whole(full[-1]) not in done:
            for q in (-1, -2):
                assert all(t[q][p] > 1.55 * min(v[p] for v in t) for p in (1, 2)), (key, t)

"""The strip kernels over device tables, as FP64 solves run them (residual with its norm,
dot product, Chebyshev steps, unconstrained products), on the grids at whose edges their
layout can go wrong: bands, blocks of node columns, planes.

A wrong residual or dot product moves the answer; a wrong smoother does not (the outer
residual corrects it) but costs iterations: the refined mode smooths with the tile kernels
and the same intervals, and its refinement only adds iterations, so FP64 may take no more
than it and two.  Bounds of the states as in test_gpu_solve.py.  Batches of different sizes
are, bit for bit, their instances alone; one has more instances than one block of flags."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import print_case

pytestmark = pytest.mark.gpu

# as in test_gpu_strips.py and test_gpu_strips_q2.py
Q1 = [(5, 5, 2), (5, 7, 2), (60, 6, 2), (61, 6, 3), (59, 6, 3), (29, 13, 2), (123, 7, 2), (14, 27, 17)]
Q2 = [(5, 3, 2), (59, 4, 2), (60, 3, 2), (61, 2, 2), (29, 8, 2), (9, 15, 9)]
CASES = [(1, n) for n in Q1] + [(2, n) for n in Q2]


def _scenario(degree, n, graded):
    s = synth.config2(ncells=n, n_steps=1)
    s.degree = degree
    if graded:
        s.edges = tuple(synth.graded_edges(0.0, s.extent[d], n[d], [(0.3 * s.extent[d], 0.6 * s.extent[d])]) for d in range(3))
    return s


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("graded", [False, True])
@pytest.mark.parametrize("degree,n", CASES, ids=["q%d %dx%dx%d" % ((d,) + n) for d, n in CASES])
def test_fp64_step_on_layout_edges(hts, degree, n, graded):
    print_case("fp64 step", degree, n, "graded", graded)
    scn = _scenario(degree, n, graded)
    Po, To, _ = oracle.run(scn, n_steps=1)
    iters = []
    for mode in (0, 1):
        o = hts.default_opts(rtol=1e-12, mode=mode)
        m = hts.from_scenario(scn, opts=o)
        _, st = m.solve_step(scn.dt, o)
        assert st["status"] == [0, 0]
        iters.append(st["iters"])
        if mode == 0:
            assert rel(m.get_state(0)[0], Po) <= 1e-10
            assert rel(m.get_state(1)[0], To) <= 1e-10
    print("iterations", iters)
    for f in (0, 1):
        assert iters[0][f] <= iters[1][f] + 2


def _alone_and_together(hts, scns, check, steps=2, **opt):
    o = hts.default_opts(**opt)
    together = [hts.from_scenario(s, opts=o) for s in scns]
    hts.advance(together, steps, scns[0].dt, o)
    for i in check:
        m = hts.from_scenario(scns[i], opts=o)
        hts.advance([m], steps, scns[i].dt, o)
        for f in (0, 1):
            assert np.array_equal(m.get_state(f)[0], together[i].get_state(f)[0]), (i, f)


@pytest.mark.parametrize("degree,sizes", [(1, Q1[2:7]), (2, Q2[1:5])], ids=["q1", "q2"])
def test_batch_of_different_sizes(hts, degree, sizes):
    print_case("fp64 batch", degree, sizes)
    scns = [_scenario(degree, n, g) for i, n in enumerate(sizes) for g in ((False, True) if i == 0 else (i % 2 == 1,))]
    _alone_and_together(hts, scns, range(len(scns)), rtol=1e-10)


@pytest.mark.parametrize("mode", [0, 1])
def test_more_instances_than_a_block_of_flags(hts, mode):
    print_case("300 instances", mode)
    scns = [_scenario(1, (4 + i % 3, 3 + i % 4, 2 + i % 2), False) for i in range(300)]
    _alone_and_together(hts, scns, (0, 1, 127, 128, 255, 256, 299), rtol=1e-10, mode=mode)

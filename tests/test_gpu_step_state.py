"""What a time step leaves behind for the next one: after a step that ran out of
iterations (its solvers stop instances and leave their flags down), after an operator
application the next step has to be, bit for bit, the one without them (both meshes have
taken a step before: the first one, also where it fails, records the spectrum behind the
heat preconditioner).  Sites with and without nodal sources (their right-hand sides end in
different kernels), node counts that end inside a block of the vector kernels."""
import numpy as np
import pytest

import synth
from gpu_util import print_case, to_dev

pytestmark = pytest.mark.gpu

SITES = [("c1", lambda: synth.config1()), ("c2", lambda: synth.config2(ncells=(17, 9, 5), n_steps=1)),
         ("c3", lambda: synth.config3(ncells=(13, 12, 7), n_steps=1))]


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("name,site", SITES, ids=[s[0] for s in SITES])
def test_a_step_after_other_calls(hts, name, site, mode, graph):
    print_case("step after other calls", name, "mode", mode, "graph", graph)
    scn = site()
    o = hts.default_opts(rtol=1e-10, mode=mode, use_graph=graph)
    short = hts.default_opts(rtol=1e-13, mode=mode, use_graph=graph, max_iter=1)
    ref, m = (hts.from_scenario(scn, opts=o) for _ in range(2))
    for k in range(2):
        ref.solve_step(scn.dt, o)
    m.solve_step(scn.dt, o)
    before = [m.get_state(f)[0] for f in (0, 1)]
    with pytest.raises(hts.HtsError):
        m.solve_step(scn.dt, short)
    for f in (0, 1):                              # nothing of it was committed
        assert np.array_equal(m.get_state(f)[0], before[f])
    x = to_dev(np.ones(m.nnode))
    y = to_dev(np.zeros(m.nnode))
    m.apply_operator(1, 0, scn.dt, x, y)
    _, st = m.solve_step(scn.dt, o)
    for f in (0, 1):
        assert np.array_equal(m.get_state(f)[0], ref.get_state(f)[0]), (f, st)

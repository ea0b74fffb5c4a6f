"""A time step does not depend on the solver mode of an earlier call: the multigrid levels
and the heat preconditioner stay with the mesh, so the smoothing intervals measured for them
have to be the same numbers whichever mode's operator kernels are in use.  After a step in
one mode and the state put back, a step in another mode is, bit for bit, the first step of
a mesh that never ran the other.  Sites with flow take the multigrid heat preconditioner
(its levels leave the convection out); sites at rest take the default one, whose interval
also holds the imaginary extent of the convection of the step that builds it."""
import numpy as np
import pytest

import synth
from gpu_util import print_case

pytestmark = pytest.mark.gpu


def _at_rest(scn):
    """The same site without flow: hydrostatic pressure, no wells.  The pressure solves of
    both modes then take no iteration and leave the same pressure."""
    scn.lines, scn.P0_steady = [], False
    scn.P0 = synth.hydrostatic(scn.extent[2], 1e5, scn.rho_w, scn.g)
    scn.bcs = [b for b in scn.bcs if b.field == 1] + [synth.FaceBC(0, f, synth.DIRICHLET, scn.P0) for f in (0, 1)]
    scn.T0 = synth.timefn(280.0, 0.05, 0.0, 0.0)
    return scn


SITES = [("q1 aquifer", lambda: synth.config2(ncells=(37, 21, 14), n_steps=1), 0),
         ("q1 piles at rest", lambda: _at_rest(synth.config3(ncells=(33, 30, 17), n_steps=1)), 1),
         ("q1 aquifer, larger", lambda: synth.config2(ncells=(65, 43, 21), n_steps=1), 0),
         ("q2 island", lambda: synth.island(ncells=(21, 13, 7), n_steps=1, degree=2), 0),
         ("q2 piles at rest", lambda: _at_rest(synth.config3(degree=2, ncells=(17, 15, 9), n_steps=1)), 1)]


@pytest.mark.parametrize("first,second", [(0, 1), (1, 0)], ids=["fp64 first", "refined first"])
@pytest.mark.parametrize("name,site,prec", SITES, ids=[s[0] for s in SITES])
def test_a_step_after_one_in_another_mode(hts, name, site, prec, first, second):
    print_case("mixed modes", name, first, second)
    scn = site()
    o1, o2 = (hts.default_opts(rtol=1e-9, mode=k, heat_precond=prec) for k in (first, second))
    ref, m = (hts.from_scenario(scn, opts=o2) for _ in range(2))
    start = [m.get_state(f)[0] for f in (0, 1)]
    _, s1 = m.solve_step(scn.dt, o1)
    for f in (0, 1):
        m.set_state(f, start[f], scn.t0)
    _, s2 = m.solve_step(scn.dt, o2)
    _, sr = ref.solve_step(scn.dt, o2)
    assert max(sr["iters"]) > 0
    assert s2["iters"] == sr["iters"]
    for f in (0, 1):
        assert np.array_equal(m.get_state(f)[0], ref.get_state(f)[0]), (f, s1, s2, sr)

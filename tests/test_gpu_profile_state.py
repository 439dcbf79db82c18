"""sphx_profile leaves the run as it was: the lists are the same after it and
an advance that follows gives the bits it gives without it, whatever the
profiled launches moved (twenty acoustic sub-steps, enough to change the
lists); a case in error keeps its lists and its error."""
import numpy as np
import pytest

from paper_2010_12375_amd import sphx
from paper_2010_12375_amd import workloads as wl
from parity import developed_state

pytestmark = pytest.mark.gpu


def lists(g, case=0):
    return [a for kind in (sphx.SPHX_INNER, sphx.SPHX_CONTACT) for a in g.get_neighbors(kind, case=case)]


@pytest.mark.parametrize("steps_before", [0, 2])
@pytest.mark.parametrize("precision", [sphx.SPHX_FP64, sphx.SPHX_FP32])
@pytest.mark.parametrize("name", ["dam2d", "sloshing", "dam3d"])
def test_a_run_goes_on_as_without_it(name, precision, steps_before):
    case = {"dam2d": lambda: wl.dam_break_2d(0.05, seed=1, precision=precision),
            "sloshing": lambda: wl.sloshing_2d(0.05, seed=1, roll=0.05, precision=precision),
            "dam3d": lambda: wl.dam_break_3d(0.1, seed=1, precision=precision)}[name]()
    state = developed_state(case, seed=4)
    sims = [sphx.Simulation.from_case(case, precision) for _ in range(2)]
    for g in sims:
        g.set_fluid(case.fluid_pos, *state)
        g.build_neighbors()
        g.advance(steps_before)
    before = lists(sims[0])
    ms = sims[0].profile(20)
    assert all(v > 0 for v in ms.values())
    for a, b in zip(before, lists(sims[0])):
        assert np.array_equal(a, b)
    for g in sims:
        g.advance(3)
    for which in range(5):
        assert np.array_equal(sims[0].get_field(which), sims[1].get_field(which)), which
    for a, b in zip(lists(sims[0]), lists(sims[1])):
        assert np.array_equal(a, b)
    for g in sims:
        g.close()


@pytest.mark.parametrize("precision", [sphx.SPHX_FP64, sphx.SPHX_FP32])
def test_a_case_in_error_keeps_its_lists(precision):
    cases = [wl.dam_break_2d(0.1, seed=k, precision=precision) for k in range(2)]
    g = sphx.Simulation.from_cases(cases, precision)
    states = [list(developed_state(c, seed=k)) for k, c in enumerate(cases)]
    # a particle that leaves the box within the first steps
    cases[1].fluid_pos[-1] = (2.0, cases[1].hi[1] - 0.01)
    states[1][0][-1] = (0.0, 50.0)
    for k, c in enumerate(cases):
        g.set_fluid(c.fluid_pos, *states[k], case=k)
    with pytest.raises(sphx.SphxError):
        g.advance(4)
    assert g.case_status(1) == sphx.SPHX_EESCAPE and g.case_status(0) == sphx.SPHX_OK
    before = [lists(g, k) for k in range(2)]
    try:
        g.profile(20)
    except sphx.SphxError:
        pass  # the launches on the case in error may raise their own
    for k in range(2):
        for a, b in zip(before[k], lists(g, k)):
            assert np.array_equal(a, b)
    assert g.case_status(1) == sphx.SPHX_EESCAPE and g.case_status(0) == sphx.SPHX_OK
    g.close()

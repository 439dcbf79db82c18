"""The wavefront-wide 3D FP64 list build where its callers and its inner path
change: the list layouts of 4, 8 and 16 lanes, several cases in one context,
walls that move beside it, and a check of the hits in the middle of a range.
Lists equal to the FP64 oracle's, rates within 1e-9 of it (the bar of every
FP64 case), a case in a batch to the bit as alone."""
import numpy as np
import pytest

import oracle as O
from paper_2010_12375_amd import sphx
from paper_2010_12375_amd import workloads as wl
from parity import developed_state, make_pair, rate_errors
from test_gpu_edge_cases import case_from, lists_equal
from test_gpu_ensemble import lists_match, snapshot

pytestmark = pytest.mark.gpu

FP64 = sphx.SPHX_FP64


def batch():
    cases = [wl.dam_break_3d(0.1, seed=3, W=0.8, precision=FP64), wl.dam_break_3d(0.15, seed=4, W=1.5, precision=FP64),
             wl.dam_break_3d(0.1, seed=5, L=0.7, H=0.5, W=0.9, precision=FP64)]
    return cases, [developed_state(c, seed=k + 1) for k, c in enumerate(cases)]


@pytest.mark.parametrize("lanes", [4, 8, 16])
def test_list_layouts_in_a_batch(lanes):
    cases, states = batch()
    g = sphx.Simulation.from_cases(cases, FP64)
    g.set_lanes(lanes)
    for k, (c, st) in enumerate(zip(cases, states)):
        g.set_fluid(c.fluid_pos, *st, case=k)
    g.build_neighbors()
    for k, (c, st) in enumerate(zip(cases, states)):
        o = O.Oracle(c)
        o.set_fluid(c.fluid_pos, *st)
        o.build_config()
        assert lists_match(g, k, o, sphx.SPHX_INNER) and lists_match(g, k, o, sphx.SPHX_CONTACT)
        _, dt = o.time_steps()
        ag, dg = g.compute_rates(dt, case=k)
        ao, do = o.compute_rates(dt)
        ea, ed = rate_errors(ag, ao, dg, do)
        print(lanes, k, c.n_fluid, "max err a", ea.max(), "drho", ed.max(), flush=True)
        assert ea.max() <= 1e-9 and ed.max() <= 1e-9
        o.close()
    g.advance(3)
    for k, (c, st) in enumerate(zip(cases, states)):
        s = sphx.Simulation.from_case(c, FP64)
        s.set_lanes(lanes)
        s.set_fluid(c.fluid_pos, *st)
        s.advance(3)
        assert snapshot(s, 0) == snapshot(g, k)
        s.close()
    g.close()


@pytest.mark.parametrize("lanes", [4, 8, 16])
def test_lists_after_the_walls_moved(lanes):
    case = wl.sloshing_3d(0.1, W=0.8, precision=FP64)
    g, o = make_pair(case, FP64)
    g.set_lanes(lanes)
    g.advance(100000, 0.2)
    while o.t < 0.2:
        o.advance(0.2)
    assert lists_equal(g, o)
    g.close()


@pytest.mark.parametrize("precision", [FP64, sphx.SPHX_FP32])
def test_hits_checked_before_the_candidates_end(precision):
    """A particle's hits are checked before all candidates are seen once they
    pass 152 - 64 = 88: here 110 in the particles' own row of cells, then more
    than two full sets of 64 candidates in later rows, all beyond 2h of them."""
    cut = 2.6 * 0.1
    rng = np.random.Generator(np.random.PCG64(14))
    tight = np.array([2.3, 2.4, 2.0]) + rng.uniform(0, 1, (110, 3)) * [0.3, 0.2, 0.1]
    far = np.array([2.0, 1.0, 3.2]) + rng.uniform(0, 1, (180, 3)) * [0.95, 2.95, 0.75]
    gap = np.linalg.norm(tight[:, None] - far[None], axis=2).min()
    # `far` lies in the rows above the cluster's cell, in its own x cell: no
    # sub-bin is trimmed, every one is a candidate
    assert gap > 1.0 and (tight.astype(int) == 2).all() and len(far) > 128
    assert ((far.astype(int) - 2 >= [0, -1, 1]) & (far.astype(int) - 2 <= [0, 1, 1])).all()
    pos = cut * np.concatenate([tight, far])
    case = case_from(pos, lo=(0.0, 0.0, 0.0), hi=(5 * cut * (1 + 1e-12),) * 3)  # five cells of 2h
    g, o = make_pair(case, precision)
    g.build_neighbors()
    o.build_config()
    assert np.diff(o.neighbors(0)[0])[:110].min() == 109
    assert lists_equal(g, o)
    g.close()

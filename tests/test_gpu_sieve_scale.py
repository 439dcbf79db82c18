"""The 3D FP64 lists at extreme units of length and in boxes smaller than the
cutoff: the first stage of the search works in FP32 and has to let every pair
within 2h through at any scale. Whole numbers, equal to the oracle's."""
import numpy as np
import pytest

from paper_2010_12375_amd import sphx
from parity import make_pair
from test_gpu_edge_cases import case_from, lists_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1e-40, 1e-20, 1e-14, 1.0, 1e14, 1e20, 1e40])
def test_lists_at_any_unit_of_length(scale):
    dp = 0.1 * scale
    cut = 2.6 * dp
    box = np.array([4.1 * cut, 4.3 * cut, 3.1 * cut])
    pos = np.random.Generator(np.random.PCG64(8)).uniform(0, 1, (700, 3)) * box
    case = case_from(pos, dp=dp, lo=(0.0, 0.0, 0.0), hi=tuple(box), periodic=(1, 0, 1))
    g, o = make_pair(case, sphx.SPHX_FP64)
    g.build_neighbors()
    o.build_config()
    assert lists_equal(g, o)
    assert np.diff(o.neighbors(0)[0]).max() > 20
    g.close()


@pytest.mark.parametrize("side", [0.3, 0.7, 0.99])
def test_lists_in_a_box_smaller_than_the_cutoff(side):
    dp = 0.1
    box = np.full(3, side * 2.6 * dp)
    pos = np.random.Generator(np.random.PCG64(9)).uniform(0, 1, (100, 3)) * box
    case = case_from(pos, dp=dp, lo=(0.0, 0.0, 0.0), hi=tuple(box))
    g, o = make_pair(case, sphx.SPHX_FP64)
    g.build_neighbors()
    o.build_config()
    assert lists_equal(g, o)
    g.close()

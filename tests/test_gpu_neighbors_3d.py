"""The 3D neighbour lists where the build's work split changes: units of
eight particles partly filled, in one cell and over many rows of cells,
stencils cut at a face and wrapped over three and more periodic cells, pairs
at the cutoff itself, more hits of one particle than are kept between two
checks. The lists are whole numbers: equal to the FP64 oracle's, both
precisions."""
import numpy as np
import pytest

from paper_2010_12375_amd import sphx
from parity import make_pair
from test_gpu_edge_cases import case_from, lists_equal

pytestmark = pytest.mark.gpu

DP = 0.1
CUT = 2.6 * DP  # 2h


def grid(counts, d):
    return np.stack(np.meshgrid(*[d * (np.arange(n) + 0.5) for n in counts], indexing="ij"), -1).reshape(-1, 3)


def walls_of(box):
    """A floor and a side of the box, half a spacing outside the fluid's range."""
    nx, ny, nz = (int(b / DP) for b in box)
    floor = grid((nx, ny, 1), DP) * [1, 1, 0] + [0, 0, 1e-3]
    side = grid((1, ny, nz), DP) * [0, 1, 1] + [1e-3, 0, 0]
    pos = np.concatenate([floor, side])
    return pos, np.concatenate([np.tile([0.0, 0, 1], (len(floor), 1)), np.tile([1.0, 0, 0], (len(side), 1))])


def positions(kind, rng):
    """Fluid, box and periodic axes of a configuration."""
    if kind.startswith("block"):  # first n sites of a jittered lattice
        n = int(kind.split("_")[1])
        return 0.1 + grid((6, 5, 5), DP)[:n] + rng.uniform(-0.02, 0.02, (n, 3)), (1.4, 1.2, 1.1), (0, 0, 0)
    if kind == "cutoff":  # distances of one and two cell sizes, up to rounding
        return grid((8, 8, 6), 0.5 * CUT), (8 * 0.5 * CUT, 8 * 0.5 * CUT, 6 * 0.5 * CUT), (1, 0, 1)
    if kind == "cluster":  # 110 particles in reach of each other around a cell corner, beside a block
        c = 2 * CUT + rng.uniform(-0.07, 0.07, (110, 3))
        return np.concatenate([c, 0.8 + grid((3, 3, 3), DP)]), (5 * CUT, 5 * CUT, 5 * CUT), (0, 0, 0)
    if kind == "sparse":  # about one particle in three cells
        box = np.array([12 * CUT, 9 * CUT, 6 * CUT])
        return rng.uniform(0, 1, (216, 3)) * box, tuple(box), (1, 1, 1)
    box = np.array([3 * CUT, 4.3 * CUT, 3 * CUT])  # "dense": three wrapped cells across
    return rng.uniform(0, 1, (900, 3)) * box, tuple(box), (1, 1, 1)


@pytest.mark.parametrize("precision", [sphx.SPHX_FP64, sphx.SPHX_FP32])
@pytest.mark.parametrize("kind", ["block_1", "block_7", "block_9", "block_64", "block_130", "cutoff", "cluster",
                                  "sparse", "dense"])
def test_lists_equal_the_oracle(kind, precision):
    pos, box, periodic = positions(kind, np.random.Generator(np.random.PCG64(5)))
    walls = None if any(periodic) else walls_of(box)
    case = case_from(pos, dp=DP, lo=(0.0, 0.0, 0.0), hi=box, walls=walls, periodic=periodic)
    g, o = make_pair(case, precision)
    g.build_neighbors()
    o.build_config()
    assert lists_equal(g, o)
    most = np.diff(o.neighbors(0)[0]).max()
    print(kind, len(pos), "particles, at most", most, "neighbours", flush=True)
    assert kind != "cluster" or most > 100
    g.close()

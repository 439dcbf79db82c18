"""The surrogate beyond 2^24 particle slots, where the byte offset of a node's
row leaves 32 bits: each particle's prediction and the gradients are those of
a small context that holds one copy of every kind of cluster."""
import numpy as np
import pytest

from paper_2010_12375_amd import gnn_inputs as gi
from paper_2010_12375_amd import sphx
from paper_2010_12375_amd import workloads as wl

pytestmark = pytest.mark.gpu

KINDS = 5  # clusters k and k + 2^22 (rows r and r + 2^24) are of different kinds
SIZE = 4


def clusters(nx, ny):
    """nx x ny clusters of four fluid particles and a wall particle, two cells
    of size 2h = 1 apart (out of reach of each other), in cell order; their
    coordinates are exact, so clusters of a kind agree to the bit."""
    rng = np.random.Generator(np.random.PCG64(12))
    off = np.array([[0.25, 0.25], [0.375, 0.25], [0.25, 0.5], [0.5, 0.375]])
    vel = rng.uniform(-0.5, 0.5, (KINDS, SIZE, 2))
    rho = 1.0 + rng.uniform(0.0, 0.01, (KINDS, SIZE))
    target = rng.normal(0, 1, (KINDS, SIZE, 3))
    n = nx * ny
    kind = np.arange(n) % KINDS
    base = 2.0 * np.stack([np.arange(n) % nx, np.arange(n) // nx], 1)
    pos = (base[:, None] + off).reshape(-1, 2)
    case = wl.Case(name="clusters", dim=2, dp=0.5, h=0.5, rho0=1.0, c0=10.0, u_ref=1.0, cfl_ad=0.25, cfl_ac=0.6,
                   gravity=(0.0, -1.0, 0.0), lo=(0.0, 0.0, 0.0), hi=(2.0 * nx, 2.0 * ny, 0.0), periodic=(0, 0, 0),
                   fluid_pos=pos, wall_pos=base + [0.375, 0.625], wall_normal=np.tile([0.0, -1.0], (n, 1)),
                   column=(1.0, 1.0))
    s = sphx.Simulation.from_case(case, sphx.SPHX_FP32)
    s.set_fluid(pos, vel[kind].reshape(-1, 2), rho[kind].reshape(-1))
    s.build_neighbors()
    c = s.counts()
    assert c["inner_pairs"] == n * SIZE * (SIZE - 1) and c["contact_pairs"] == n * SIZE
    s.gnn_set_params(gi.init_params(31))
    return s, kind, target[kind].reshape(-1, 3)


def test_rows_beyond_32_bit_offsets():
    few, _, target = clusters(KINDS, 1)
    few.gnn_forward()
    expect = few.gnn_output().reshape(KINDS, SIZE, 3)
    few.gnn_set_target(target)
    loss = few.gnn_train_step(1e-3)
    grad = gi.unpack(few.gnn_get_grad().astype(np.float64))
    few.close()
    many, kind, target = clusters(2048, 2112)
    assert len(target) > (1 << 24) + (1 << 18)
    many.gnn_forward()
    out = many.gnn_output().reshape(-1, SIZE, 3)
    for k in range(KINDS):
        assert (out[kind == k] == expect[k]).all(), k
    many.gnn_set_target(target)
    # the means are over the kinds in nearly equal parts (2^22 + 2^17 clusters:
    # 1e-6); a sum of up to n = 17 408 FP32 terms in a chain (rows of a block,
    # then blocks) is off by at most n 2^-24 of its terms' absolute sum, for
    # which sixteen times the result is allowed
    tol = 16 * 17408 * 2.0 ** -24
    assert abs(many.gnn_train_step(1e-3) - loss) <= 1e-5 * loss
    got = gi.unpack(many.gnn_get_grad().astype(np.float64))
    many.close()
    for name, g in grad.items():
        assert np.linalg.norm(got[name] - g) <= tol * np.linalg.norm(g) + 1e-12, name

"""The surrogate's inference kernels at the sizes and layouts where their
launch shape changes: 16 or 32 nodes per block (the larger batch takes 32),
list layouts of 2, 4 and 8 lanes, isolated particles and particles with wall
edges only, FP32 and FP64 state."""
import math

import numpy as np
import pytest

from oracle import gnn_oracle as G
from paper_2010_12375_amd import gnn_inputs as gi
from paper_2010_12375_amd import sphx
from paper_2010_12375_amd import workloads as wl
from parity import developed_state
from test_gpu_surrogate import assert_outputs_match, gpu_sim, oracle_forward

pytestmark = pytest.mark.gpu


def test_wide_batch_equals_single_cases():
    """Six cases of 12 800 particles (32 nodes per block) give each case the
    bits it has alone (16 per block): no sum depends on the launch shape."""
    cases = [wl.dam_break_2d(0.0125, seed=k, L=math.sqrt(2 / a), H=math.sqrt(2 * a), precision=sphx.SPHX_FP32)
             for k, a in enumerate((0.25, 0.4, 0.55, 0.7, 0.85, 1.0))]
    states = [developed_state(c, seed=k) for k, c in enumerate(cases)]
    params = gi.init_params(21)
    b = gpu_sim(cases, states, sphx.SPHX_FP32, params)
    b.gnn_forward()
    outs = [b.gnn_output(case=k) for k in range(len(cases))]
    b.close()
    assert sum(c.n_fluid for c in cases) > 1 << 16
    for k in (0, 3, 5):
        s = gpu_sim([cases[k]], [states[k]], sphx.SPHX_FP32, params)
        s.gnn_forward()
        assert np.array_equal(s.gnn_output(), outs[k])
        s.close()


@pytest.mark.parametrize("precision", [sphx.SPHX_FP32, sphx.SPHX_FP64])
@pytest.mark.parametrize("lanes", [2, 4, 8])
def test_list_layouts(lanes, precision):
    case = wl.config_small(3)
    st = developed_state(case, seed=3)
    params = gi.init_params(22)
    _, Yo, _ = oracle_forward(case, st, params)
    s = gpu_sim([case], [st], precision, params)
    s.set_lanes(lanes)
    s.gnn_forward()
    assert_outputs_match(s.gnn_output(), Yo, f"{lanes} lanes")
    s.close()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 65])
def test_few_and_isolated_particles(n):
    """n particles in a row one spacing apart, every fifth lifted out of
    reach of all others: nodes without edges, nodes with wall edges only."""
    case = wl.config_small(4)
    dp = case.dp
    x = np.column_stack([(np.arange(n) + 0.5) * dp, np.full(n, 0.5 * dp)])
    x[4::5, 1] = 1.0 + 6 * dp * np.arange(len(x[4::5])) / max(1, len(x[4::5]))
    case.fluid_pos = x
    st = developed_state(case, seed=4)
    params = gi.init_params(23)
    _, Yo, _ = oracle_forward(case, st, params)
    s = gpu_sim([case], [st], sphx.SPHX_FP32, params)
    s.gnn_forward()
    rms = float(np.sqrt((Yo ** 2).mean()))
    # one rounding flip moves an output by about 2^-8 of itself (test_gpu_surrogate.py)
    assert np.abs(s.gnn_output() - Yo).max() <= 8 * 2.0 ** -8 * rms
    s.close()


def _row(n):
    case = wl.config_small(5)
    dp = case.dp
    x = np.column_stack([(np.arange(n) + 0.5) * dp, np.full(n, 0.5 * dp)])
    x[4::5, 1] = 1.0 + 0.5 * np.arange(len(x[4::5]))[: len(x[4::5])] % 4.0
    case.fluid_pos = x
    return case


@pytest.mark.parametrize("case,tol", [(_row(3), 8 * 2.0 ** -8), (_row(65), 8 * 2.0 ** -8),
                                      (wl.dam_break_2d(0.0115, seed=6, precision=sphx.SPHX_FP32), 5e-3)],
                         ids=["3", "65", "15k"])
def test_training_gradients_at_ragged_sizes(case, tol):
    """Edge counts below one step of 64, not a multiple of it, and beyond 256
    rows a block (there: 320, a half step at the end). Tolerances: one
    rounding flip (8 x 2^-8, test_gpu_surrogate.py) where a tensor's norm
    comes from few particles, that file's 5e-3 at 15 000."""
    st = developed_state(case, seed=6)
    params = gi.init_params(24)
    T = np.random.Generator(np.random.PCG64(98)).normal(0, 1, (case.n_fluid, 3))
    g, Yo, cache = oracle_forward(case, st, params)
    _, dY = G.loss_grad(Yo, T)
    grad_o = G.backward(params.astype(np.float64), g, cache, dY, emu=True)
    s = gpu_sim([case], [st], sphx.SPHX_FP32, params)
    s.gnn_set_target(T)
    s.gnn_train_step(1e-3)
    pg, names = G.unpack(s.gnn_get_grad().astype(np.float64))
    po, _ = G.unpack(grad_o)
    s.close()
    for n in names:
        assert np.linalg.norm(pg[n] - po[n]) <= tol * np.linalg.norm(po[n]) + 1e-12, n

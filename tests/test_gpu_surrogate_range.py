"""The surrogate's layers where a tile of edges is only partly filled and the
message inputs are near the largest FP32 value: the places without an edge
add nothing, whatever the sums at the others."""
import numpy as np
import pytest

from paper_2010_12375_amd import gnn_inputs as gi
from paper_2010_12375_amd import sphx
from paper_2010_12375_amd import workloads as wl
from parity import developed_state
from test_gpu_surrogate import gpu_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("train", [False, True])
def test_places_without_an_edge_add_nothing(train):
    """Pairs of particles with one edge each. With the messages' share of the
    update at zero, message biases of 3.2e38 (sums of one message are finite)
    change no output and no loss."""
    case = wl.config_small(5)
    dp = case.dp
    x = np.array([[0.5 + 8 * dp * k + dp * i, 3.0] for k in range(5) for i in range(2)])
    case.fluid_pos = x
    st = developed_state(case, seed=5)
    T = np.random.Generator(np.random.PCG64(3)).normal(0, 1, (len(x), 3))
    got = []
    for bias in (0.0, 3.2e38):
        params = gi.init_params(25)
        v = gi.unpack(params)
        for l in range(gi.LAYERS):
            v[f"Wu{l}"][gi.HIDDEN:] = 0.0
            v[f"bm{l}"][:] = bias
        s = gpu_sim([case], [st], sphx.SPHX_FP32, params)
        assert s.counts()["inner_pairs"] == len(x) and s.counts()["contact_pairs"] == 0
        if train:
            s.gnn_set_target(T)
            got.append(s.gnn_train_step(1e-3))
        else:
            s.gnn_forward()
            got.append(s.gnn_output())
        s.close()
    assert np.isfinite(got[0]).all()
    assert np.array_equal(got[0], got[1])

"""Fields read to device memory, written by the kernel where it can and copied
where it cannot (an address that is not a multiple of eight): the values of
the host read, and nothing beside them."""
import numpy as np
import pytest
import torch

from paper_2010_12375_amd import sphx
from paper_2010_12375_amd import workloads as wl
from parity import developed_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("byte_offset", [0, 8, 4])
@pytest.mark.parametrize("dim,precision", [(2, sphx.SPHX_FP32), (2, sphx.SPHX_FP64), (3, sphx.SPHX_FP32)])
def test_device_read_equals_host_read(dim, precision, byte_offset):
    if dim == 2:
        case = wl.dam_break_2d(0.1, precision=precision)
    else:
        case = wl.dam_break_3d(0.2, W=2.0, precision=precision)
    vel, rho, drho = developed_state(case, seed=2)
    g = sphx.Simulation.from_case(case, precision)
    g.set_fluid(case.fluid_pos, vel, rho, drho)
    g.advance(2)
    n = case.n_fluid
    for which in range(5):
        ref = g.get_field(which)
        raw = torch.full((ref.size * 8 + 64,), 0x5A, dtype=torch.uint8, device="cuda:0")
        torch.cuda.synchronize()
        g.get_field_device(which, raw.data_ptr() + byte_offset)
        got = raw.cpu().numpy()
        body = got[byte_offset:byte_offset + ref.size * 8].copy().view(np.float64).reshape(ref.shape)
        assert np.array_equal(body, ref), which
        assert (got[:byte_offset] == 0x5A).all() and (got[byte_offset + ref.size * 8:] == 0x5A).all()
    assert n > 64
    g.close()

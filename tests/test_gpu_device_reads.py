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


@pytest.mark.parametrize("byte_offset", [0, 8, 4])
@pytest.mark.parametrize("given", ["all", "pos_rho", "pos"])
@pytest.mark.parametrize("dim,precision", [(2, sphx.SPHX_FP64), (3, sphx.SPHX_FP32)])
def test_device_set_equals_host_set(dim, precision, given, byte_offset):
    """Fluid set from device memory, read in place or copied, continues as
    the same arrays set from the host."""
    case = wl.dam_break_2d(0.1, precision=precision) if dim == 2 else wl.dam_break_3d(0.2, W=2.0, precision=precision)
    vel, rho, drho = developed_state(case, seed=3)
    arrays = {"all": (vel, rho, drho), "pos_rho": (None, rho, None), "pos": (None, None, None)}[given]
    arrays = (case.fluid_pos,) + arrays
    sims = [sphx.Simulation.from_case(case, precision) for _ in range(2)]
    for g in sims:
        g.advance(1)  # laid out: the next set is from the device arrays themselves
    kept, ptrs = [], []
    for a in arrays:
        if a is None:
            ptrs.append(None)
            continue
        raw = torch.zeros(a.size * 8 + 16, dtype=torch.uint8)
        raw[byte_offset:byte_offset + a.size * 8] = torch.from_numpy(np.ascontiguousarray(a).reshape(-1).view(np.uint8))
        kept.append(raw.to("cuda:0"))
        ptrs.append(kept[-1].data_ptr() + byte_offset)
    torch.cuda.synchronize()
    sims[0].set_fluid(*arrays)
    sims[1].set_fluid_device(case.n_fluid, *ptrs)
    for g in sims:
        g.advance(3)
    for which in range(5):
        assert np.array_equal(sims[0].get_field(which), sims[1].get_field(which)), which
    for g in sims:
        g.close()

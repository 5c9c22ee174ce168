"""Readback of fields, spectra and gradients (fdtd_get_field, fdtd_monitor_dft,
fdtd_get_grad) through the pinned ring: the bytes are those of the device
arrays, at row lengths that leave every remainder of a 16-byte store, at sizes
below one slot, of whole slots, around the eight slots of the ring, and at and
above the 4 MiB from which helper threads copy."""
import numpy as np
import pytest

from paper_2609_30039_amd import binding as B
from paper_2609_30039_amd import workloads
from paper_2609_30039_amd.sim import Simulation

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,dtype", [
    ((3, 3, 3), "f32"), ((5, 7, 9), "f64"), ((66, 31, 13), "f32"), ((64, 64, 64), "f32"), ((64, 64, 32), "f64"),
    ((64, 64, 65), "f32"), ((127, 129, 64), "f32"), ((128, 128, 64), "f32"), ((201, 203, 105), "f32"),
    ((131, 137, 149), "f64"),
])
def test_field_readback_returns_the_uploaded_bytes(shape, dtype):
    nx, ny, nz = shape
    spec = workloads.DomainSpec(shape=shape, courant=0.5, n_steps=1)
    sim = Simulation(spec, dtype=dtype)
    rng = np.random.default_rng(nx * ny + nz)
    want = [rng.standard_normal((nz, ny, nx)).astype(sim.dtype) for _ in range(3)]
    want[1][0, 0, 0] = -0.0
    want[2][-1, -1, -1] = np.inf
    for c in range(3):
        sim.set_field(2 * c, want[c])
    for _ in range(2):   # a used ring as well as a fresh one
        for c in range(3):
            got = sim.field(2 * c)
            assert got.tobytes() == want[c].tobytes()
    # an unaligned destination inside a larger buffer, its neighbours untouched
    es = want[0].itemsize
    raw = np.full(want[0].nbytes + 3 * es, 0x5A, dtype=np.uint8)
    out = np.frombuffer(raw.data, dtype=sim.dtype, count=want[0].size, offset=es)
    B.fdtd_get_field(sim.h, 0, 0, out)
    assert out.tobytes() == want[0].tobytes()
    assert np.all(raw[:es] == 0x5A) and np.all(raw[es + want[0].nbytes:] == 0x5A)
    with pytest.raises(B.FdtdError):   # one element short: refused, nothing written
        B.fdtd_get_field(sim.h, 0, 0, np.empty(want[0].size - 1, dtype=sim.dtype))
    sim.close()

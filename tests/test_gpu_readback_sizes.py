"""Reads of contiguous fields on either side of the sizes at which a handle takes
the runtime's copy or its pinned ring, the first reads and later ones, with a
pitched read between them."""
import numpy as np
import pytest

from paper_2609_30039_amd import workloads as W
from paper_2609_30039_amd.sim import Simulation

pytestmark = pytest.mark.gpu

KI = 1024


@pytest.mark.parametrize("kib", [2, 256, 258, 2046, 2048, 2050, 8190, 8192, 8194])
def test_contiguous_reads(kib):
    rows = kib * KI // 128   # 16 FP64 cells: a pitch
    ny = 2 if rows % 2 == 0 else 1
    spec = W.DomainSpec(shape=(16, ny, rows // ny), courant=W.courant_3d(), n_steps=1)
    odd = W.DomainSpec(shape=(5, 3, 7), courant=W.courant_3d(), n_steps=1)
    rng = np.random.default_rng(kib)
    sim = Simulation([spec, odd], dtype="f64", max_steps=1)
    want = rng.standard_normal((rows // ny, ny, 16))
    small = rng.standard_normal((7, 3, 5))
    for read in range(7):
        sim.set_field(3, want + read, 0)
        if read == 5:
            sim.set_field(4, small, 1)
            assert np.array_equal(sim.field(4, 1), small)
        assert np.array_equal(sim.field(3, 0), want + read), read
    sim.close()

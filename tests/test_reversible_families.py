"""Kernel families in the reversible mode: every launch shape that the autotuner
can return for such a domain is admitted, and the families give the same bits."""
import numpy as np
import pytest

from paper_2609_30039_amd import adjoint as A
from paper_2609_30039_amd import autotune as AT
from paper_2609_30039_amd import binding as B
from paper_2609_30039_amd import workloads as W
from paper_2609_30039_amd.sim import Simulation

N = 40


def _spec(shape=(70, 34, 38)):
    return W.design_patch(pml=6, design=12, patch=10, n_steps=N, n_f=2, shape=shape)[0]


@pytest.mark.parametrize("cand", AT.CANDIDATES, ids=lambda c: "{kernel}-{tile_rows}-{tile_kz}".format(**c))
def test_tuned_shapes_are_admitted(cand):
    """Validation passes; the tiny budget refuses afterwards."""
    kern = {"split": B.FDTD_KERNEL_SPLIT, "onepass": B.FDTD_KERNEL_ONEPASS, "fused": B.FDTD_KERNEL_FUSED}[cand["kernel"]]
    with pytest.raises(B.FdtdError) as e:
        B.fdtd_create([_spec()], B.FDTD_F32, kernel=kern, tile_rows=cand["tile_rows"], tile_kz=cand["tile_kz"],
                      max_steps=N, reversible=True, mem_budget_bytes=1.0)
    assert e.value.code == B.FDTD_E_NOMEM


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("kw", [dict(kernel="onepass"), dict(kernel="onepass", tile_kz=16),
                                dict(kernel="onepass", tile_rows=8, tile_kz=64), dict()],
                         ids=["onepass", "onepass-16", "onepass-8-64", "auto"])
def test_reversible_families_bitwise(kw, dtype):
    """A batch of two domains, forward with the interface recorded, reverse:
    fields, spectra and gradients of the split kernels."""
    def run(**k):
        specs = [_spec(), _spec((41, 36, 37))]
        sim = Simulation(specs, dtype=dtype, reversible=True, max_steps=N, **k)
        g = A.reversible_gradient(sim, N, lambda s: {(d, 0): 2.0 * s.spectra(0, d) for d in range(2)})
        out = list(g) + [sim.spectra(0, d) for d in range(2)]
        out += [sim.field(q, d, adjoint=True) for d in range(2) for q in range(6)]
        sim.close()
        return out

    for q, (x, y) in enumerate(zip(run(kernel="split"), run(**kw))):
        assert np.array_equal(x, y), (q, np.abs(x - y).max())
        assert np.abs(x).max() > 0

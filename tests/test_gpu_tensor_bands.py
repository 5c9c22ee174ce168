"""Tensor adjoint nodes at the edges of their bands: planes of one band of 128
blocks, of one block more (two bands, the last one with an empty block) and of
three bands; the gradient against the oracle's transposed sweep with a source
sheet and a point beside a band's edge."""
import numpy as np
import pytest

from paper_2609_30039_amd import workloads as W
from tests.gpu_util import gpu_gradient_store_all, oracle_gradient, rel
from tests.test_gpu_tensor_nodes import _cot

pytestmark = pytest.mark.gpu


# the bars of the tensor gradient elsewhere: FP64 round-off, FP32 by its rounding order
@pytest.mark.parametrize("dtype,tol", [("f64", 1e-11), ("f32", 2e-5)])
@pytest.mark.parametrize("shape,pml", [((256, 128, 4), (0,) * 6), ((257, 128, 5), (2, 0, 0, 2, 0, 0)), ((330, 201, 3), (0,) * 6)])
def test_tensor_gradient_across_bands(shape, pml, dtype, tol):
    nx, ny, nz = shape
    rng = np.random.Generator(np.random.PCG64(nx))
    lo = tuple(pml[2 * a] for a in range(3))
    hi = tuple(shape[a] - pml[2 * a + 1] for a in range(3))
    b = tuple(hi[a] - lo[a] for a in (2, 1, 0))
    n = 6
    wave = W.gaussian_sine(n, 0.5, 2.0, 1.0)
    spec = W.DomainSpec(
        shape=shape, courant=W.courant_3d(), pml=pml, eps_kind="tensor", eps_box=(lo, hi),
        eps=W.random_spd_tensors(rng, b[0] * b[1] * b[2]).reshape((6,) + b), n_steps=n, grad_box=(lo, hi),
        sources=[W.SourceSpec("plane_z", 0, (0, 0, 1), wave), W.SourceSpec("point", 2, (nx // 2, ny // 2, nz // 2), wave)],
        monitors=[W.MonitorSpec("patch_z", comp=0, pos=(0, 0, nz // 2), rect=(1, nx, 1, ny), omega_dt=W.freq_grid(2)),
                  W.MonitorSpec("patch_z", comp=4, pos=(0, 0, nz // 2), rect=(0, nx, 0, ny), omega_dt=W.freq_grid(1))])
    sim, g, _ = gpu_gradient_store_all(spec, dtype, _cot)
    sim.close()
    _, ref = oracle_gradient(spec, _cot)
    ref = ref[:, lo[2]:hi[2], lo[1]:hi[1], lo[0]:hi[0]]
    assert (np.abs(ref).max(axis=(0, 1, 3)) > 0).all() and g.shape == ref.shape
    assert rel(g, ref) < tol

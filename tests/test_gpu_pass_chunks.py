"""Sources beside the z cuts of long chunks: the single pass recomputes E of the
plane above a chunk, so a source there belongs to both chunks.  Explicit chunk
lengths at and above the kernel's limit, bit for bit against the split kernels."""
import numpy as np
import pytest

import test_gpu_pass as tf
from paper_2609_30039_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nz,pml", [(128, 0), (192, 0), (95, 0), (150, 0), (128, 3)])
@pytest.mark.parametrize("tile_kz", [62, 63, 64, 200])
def test_sources_on_chunk_boundaries(tile_kz, nz, pml, dtype):
    nx, ny = 23, 12
    wave = W.gaussian_sine(4, 0.4, 3.0, 2.0)
    cuts = sorted({c + o for c in (nz // 3, nz // 2, 2 * nz // 3, 62, 63, 64) for o in (0, 1)})
    for z in cuts:
        spec = tf._spec((nx, ny, nz), pml=(0, 0, 0, 0, pml, pml), n=4)
        spec.sources = [W.SourceSpec("plane_z", 0, (0, 0, z), wave), W.SourceSpec("point", 1, (nx // 2, ny // 2, z), wave),
                        W.SourceSpec("point", 2, (3, ny - 1, min(z + 1, nz - 1)), wave)]
        spec.monitors[4] = W.MonitorSpec("probe", comp=4, pos=(nx // 2, ny // 2, z - 1))   # H below the source plane
        tf._same([spec], dtype, steps=4, tile_kz=tile_kz)

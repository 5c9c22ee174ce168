"""Dispersive boxes on one side of a periodic seam, away from the last tile on
the other side: the tiles that end at the seam meet them only through their
wrapped halo.  Single-pass forward and adjoint against the split kernels, bit
for bit, with several tiles in x and in y."""
import numpy as np
import pytest

import test_gpu_adj_pass as ta
import test_gpu_pass as tf
from paper_2609_30039_amd import workloads as W

pytestmark = pytest.mark.gpu

SHAPE = (120, 48, 40)
BOXES = [((0, 0, 15), (5, 48, 25)), ((0, 0, 15), (120, 24, 25)), ((0, 3, 15), (7, 9, 25)),
         ((115, 3, 15), (120, 40, 25)), ((2, 43, 15), (119, 48, 25))]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("poles", [1, 3])
@pytest.mark.parametrize("box", range(len(BOXES)))
def test_box_beside_a_seam(box, poles, dtype):
    lo, hi = BOXES[box]
    for sign in ((1, -1, 1), (-1, 1, 1)):
        kw = dict(shape=SHAPE, pml=(0, 0, 0, 0, 6, 6), per=(1, 1, 0), sign=sign)
        lor = [W.LorentzSpec(lo, hi, 1.2, 0.35, 0.02, poles=W.pole_set(poles) if poles > 1 else None)]
        spec = tf._spec(**kw)
        spec.lorentz = lor
        tf._same([spec], dtype, steps=4)
        spec = ta._spec(**kw)
        spec.lorentz = lor
        ta._same([spec], dtype)

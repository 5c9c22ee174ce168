"""AUTO's mixed routes against the split kernels, bit for bit: single-pass forward
with the split adjoint, split forward with the single-pass adjoint, and both
split, for the dispersive domains that take them (periodic with the box in all
of it, a box on line boundaries, a box over most of a walled domain), alone and
in a batch with a domain that takes the single pass for both."""
import numpy as np
import pytest

import test_gpu_adj_pass as ta
import test_gpu_pass as tf
from paper_2609_30039_amd import workloads as W

pytestmark = pytest.mark.gpu

PER = dict(pml=(0, 0, 0, 0, 6, 6), per=(1, 1, 0), sign=(-1, 1, 1))
CASES = {   # shape, dtype, box, poles, options
    "periodic f64": ((128, 128, 132), "f64", ((0, 0, 6), (128, 128, 126)), 1, PER),
    "aligned f32": ((200, 200, 200), "f32", ((32, 32, 32), (160, 160, 160)), 6, dict(pml=(8,) * 6)),
    "walled f32": ((60, 52, 56), "f32", ((6, 6, 6), (54, 46, 50)), 3, dict(pml=(6,) * 6)),
    "walled f64": ((61, 52, 57), "f64", ((5, 6, 7), (55, 45, 51)), 1, dict(pml=(6,) * 6)),
}


def _spec(mod, name):
    shape, _, (lo, hi), poles, kw = CASES[name]
    s = mod._spec(shape, **kw)
    s.lorentz = [W.LorentzSpec(lo, hi, 1.2, 0.35, 0.02, poles=(W.pole_set(16)[:poles] if poles > 1 else None))]
    return s


@pytest.mark.parametrize("name", list(CASES))
def test_mixed_routes_bitwise(name):
    dtype = CASES[name][1]
    big = CASES[name][0][0] > 100
    if big:   # a small gradient box keeps the read small
        spec = _spec(ta, name)
        spec.grad_box = ((10, 20, 30), (60, 50, 40))
        ta._same([spec], dtype)
    else:
        other = ta._spec((49, 9, 17), pml=(3, 2, 2, 3, 5, 4))
        ta._same([_spec(ta, name)], dtype)
        ta._same([other, _spec(ta, name)], dtype)
    a, _ = tf._run([_spec(tf, name)], dtype, 4, comps=(0, 1, 5), kernel="split")
    for chunk in (0, 2):
        b, _ = tf._run([_spec(tf, name)], dtype, 4, comps=(0, 1, 5), graph_chunk=chunk)
        assert all(np.array_equal(x, y) for x, y in zip(a[:5], b[:5]))

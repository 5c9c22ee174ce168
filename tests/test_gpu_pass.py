"""The single-pass forward kernel against the split kernels, bit for bit: fields,
probe traces and spectra from random states, where its tiles, halos and
variants can go wrong: domains smaller than a tile and of one cell more than
one, odd and even rows, slabs that meet half a column group, sources and
monitors on the first and last plane, dispersive boxes in a slab and across a
seam, periodic seams, each block shape, ragged batches, captured chunks of odd
and even length, and steps from a restored slot."""
import numpy as np
import pytest

from paper_2609_30039_amd import workloads as W
from paper_2609_30039_amd.sim import Simulation

pytestmark = pytest.mark.gpu


def _spec(shape, pml=(0,) * 6, kind="iso", poles=0, per=(0, 0, 0), sign=(1, 1, 1), seed=3, n=6):
    nx, ny, nz = shape
    rng = np.random.Generator(np.random.PCG64(seed))
    lo = tuple(pml[2 * a] for a in range(3))
    hi = tuple(shape[a] - pml[2 * a + 1] for a in range(3))
    eps = 1.0 + 3.0 * rng.random((3 if kind == "diag" else 1, hi[2] - lo[2], hi[1] - lo[1], hi[0] - lo[0]))
    lor = []
    if poles:
        # reaches into the slabs and to the seams; odd start along x
        b0, b1 = (1, 1, 1), tuple(max(2, (2 * s) // 3) for s in shape)
        lor = [W.LorentzSpec(b0, b1, 1.2, 0.35, 0.02, poles=W.pole_set(poles) if poles > 1 else None)]
    wave = W.gaussian_sine(n, 0.4, 3.0, 2.0)
    return W.DomainSpec(
        shape=shape, courant=W.courant_3d(), pml=pml, eps_kind=kind, eps_box=(lo, hi), eps=eps, eps_bg=1.5,
        lorentz=lor, periodic=per, bloch_sign=sign, n_steps=n,
        sources=[W.SourceSpec("plane_z", 0, (0, 0, nz - 1), wave),
                 W.SourceSpec("point", 2, (nx - 1, ny // 2, 0), wave),
                 W.SourceSpec("point", 1, (nx // 2, ny - 1, nz // 2), wave)],
        monitors=[W.MonitorSpec("flux_z", pos=(0, 0, 0), rect=(0, nx, 0, ny), omega_dt=W.freq_grid(2)),
                  W.MonitorSpec("flux_z", pos=(0, 0, nz // 2), rect=(0, nx, 0, ny), omega_dt=W.freq_grid(2)),
                  W.MonitorSpec("patch_z", comp=5, pos=(0, 0, nz - 1), rect=(0, nx, 0, ny), omega_dt=W.freq_grid(3)),
                  W.MonitorSpec("probe", comp=4, pos=(nx - 1, ny - 1, nz - 1)),
                  W.MonitorSpec("probe", comp=2, pos=(nx // 2, ny // 2, nz // 2))])


def _run(specs, dtype, steps, comps=range(6), slot=False, **kw):
    s = Simulation(specs, dtype=dtype, max_steps=steps, n_ckpt=1 if slot else 0, **kw)
    rng = np.random.Generator(np.random.PCG64(5))
    for d, sp in enumerate(specs):
        nx, ny, nz = sp.shape
        for q in range(6):
            v = rng.standard_normal((nz, ny, nx), dtype=np.float32)
            if q < 3:   # E tangential to a wall is zero
                for a in ((q + 1) % 3, (q + 2) % 3):
                    if not sp.periodic[a]:
                        v[tuple(slice(0, 1) if 2 - a == m else slice(None) for m in range(3))] = 0
            s.set_field(q, v, d)
    if slot:
        s.step(2, record=False)
        s.save(0)
        s.step(1, record=False)
        s.restore(0)
    s.step(steps // 2)
    s.step(steps - steps // 2)
    out = []
    for d, sp in enumerate(specs):
        out += [s.field(q, d) for q in comps]
        out += [s.probe(m, d) for m, mon in enumerate(sp.monitors) if mon.kind == "probe"]
        out += [s.spectra(m, d) for m, mon in enumerate(sp.monitors) if mon.kind != "probe"]
    s.close()
    return out, len(list(comps)) + 2


def _same(specs, dtype, steps=6, chunk=0, **kw):
    a, nf = _run(specs, dtype, steps, kernel="split", **kw)
    b, _ = _run(specs, dtype, steps, kernel="onepass", graph_chunk=chunk, **kw)
    per = len(a) // len(specs)
    for q, (x, y) in enumerate(zip(a, b)):
        if q % per < nf or not chunk:
            assert np.array_equal(x, y), (q, np.abs(x - y).max())
        else:   # spectra: a chunk's samples are summed in other blocks (FP64 sums of FP32 or FP64 samples)
            assert np.abs(x - y).max() <= 1e-13 * steps * np.abs(x).max(), q


CASES = [
    dict(shape=(5, 4, 6)),
    dict(shape=(2, 3, 3), kind="diag"),
    dict(shape=(1, 1, 4)),
    dict(shape=(49, 9, 17), pml=(3, 2, 2, 3, 5, 4)),                       # odd row, half groups in the slabs
    dict(shape=(50, 10, 16), pml=(0, 3, 0, 4, 0, 5), kind="diag"),         # slabs on the high sides only
    dict(shape=(51, 8, 33), pml=(5, 0, 3, 0, 4, 0), poles=1),
    dict(shape=(97, 23, 18), pml=(4,) * 6, kind="diag", poles=1),
    dict(shape=(40, 21, 19), pml=(3,) * 6, poles=3),
    dict(shape=(33, 12, 14), pml=(2,) * 6, poles=16),
    dict(shape=(48, 7, 20), pml=(0, 0, 0, 0, 6, 6), per=(1, 1, 0), sign=(-1, 1, 1), kind="diag"),
    dict(shape=(52, 24, 15), pml=(0, 0, 4, 4, 3, 3), per=(1, 0, 0), sign=(-1, 1, 1), poles=1),
    dict(shape=(31, 9, 16), pml=(3, 3, 0, 0, 3, 3), per=(0, 1, 0), sign=(1, -1, 1), poles=3),
    dict(shape=(31, 9, 16), per=(1, 1, 0), sign=(-1, -1, 1)),              # FP32: odd periodic x stays on the split kernels
    dict(shape=(2, 2, 8), per=(1, 1, 0)),
]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_pass_equals_split_bitwise(case, dtype):
    spec = _spec(seed=case, **CASES[case])
    _same([spec], dtype, chunk=(0, 2, 3)[case % 3])
    _same([spec], dtype, tile_kz=(1, 4, 64)[case % 3])


def test_pass_from_a_slot_and_in_a_ragged_batch():
    specs = [_spec(seed=k, **CASES[k]) for k in (3, 6, 9, 12)]   # the last one split in FP32
    for dtype in ("f32", "f64"):
        _same(specs, dtype, slot=True, chunk=3)
    t = W.anisotropic_tensor(interior=12, pml=4, patch=4, n_steps=6, n_f=2)
    t.monitors += [W.MonitorSpec("probe", comp=4, pos=(3, 3, 3)), W.MonitorSpec("probe", comp=1, pos=(9, 9, 9))]
    t.monitors += [W.MonitorSpec("patch_z", comp=1, pos=(0, 0, k), rect=(0, 9, 0, 9), omega_dt=W.freq_grid(2)) for k in (5, 6)]
    _same([specs[0], t, specs[1]], "f32", chunk=3)


@pytest.mark.parametrize("shape,dtype", [((170, 161, 145), "f32"), ((262, 201, 197), "f32"), ((200, 160, 170), "f64"),
                                         ((352, 345, 347), "f32")])
def test_pass_block_shapes(shape, dtype):
    """Domains that take the 512- and the 1024-thread blocks."""
    _same([_spec(shape, pml=(7, 8, 9, 6, 5, 10), kind="diag", poles=1, n=4)], dtype, steps=4, comps=(0, 4))


def test_auto_picks_by_size_and_shape():
    """AUTO and explicit launch shapes all give the split results."""
    spec = _spec((60, 31, 26), pml=(4,) * 6, poles=1)
    ref, _ = _run([spec], "f32", 6, kernel="split")
    for kw in (dict(), dict(tile_rows=8, tile_kz=3), dict(kernel="onepass", tile_rows=4, tile_kz=200)):
        got, _ = _run([spec], "f32", 6, **kw)
        assert all(np.array_equal(a, b) for a, b in zip(ref, got)), kw

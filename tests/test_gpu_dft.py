"""The spectra of all plane monitors, summed in one launch: against the host sum
of the same samples, for frequency counts around the block's group of four,
planes of less and more than a block of points, more monitors than one launch
takes, monitors read or cleared at different steps (so that their buffered
samples differ in number), and captured chunks."""
import numpy as np
import pytest

from paper_2609_30039_amd import workloads as W
from paper_2609_30039_amd.sim import Simulation

pytestmark = pytest.mark.gpu

SHAPE = (20, 19, 8)
N = 11


def _spec(nf):
    nx, ny, nz = SHAPE
    fr = W.freq_grid(nf, 0.1, 0.6)
    mons = [W.MonitorSpec("flux_z", pos=(0, 0, 4), rect=(0, nx, 0, ny), omega_dt=fr),
            W.MonitorSpec("flux_z", pos=(0, 0, 0), rect=(3, 4, 2, 3), omega_dt=fr[:1]),
            W.MonitorSpec("patch_z", comp=2, pos=(0, 0, 5), rect=(2, 18, 1, 17), omega_dt=fr),
            W.MonitorSpec("patch_z", comp=4, pos=(0, 0, 5), rect=(0, nx, 0, ny), omega_dt=fr),
            W.MonitorSpec("patch_z", comp=0, pos=(0, 0, nz - 1), rect=(0, nx, 0, 1), omega_dt=fr)]
    return W.DomainSpec(shape=SHAPE, courant=0.5, n_steps=N, monitors=mons,
                        sources=[W.SourceSpec("point", 2, (9, 9, 4), W.gaussian_sine(N, 0.5, 3.0, 2.0))])


def _fill(sim, d):
    nx, ny, nz = SHAPE
    rng = np.random.default_rng(d)
    for q in range(6):
        v = rng.standard_normal((nz, ny, nx))
        for a in ((q + 1) % 3, (q + 2) % 3) if q < 3 else ():
            v[tuple(slice(0, 1) if 2 - a == m else slice(None) for m in range(3))] = 0
        sim.set_field(q, v, d)


def _sum(spec, hist, m, n0, dtype):
    mon = spec.monitors[m]
    i0, i1, j0, j1 = mon.rect
    k = mon.pos[2]
    comps = (0, 1, 3, 4) if mon.kind == "flux_z" else (mon.comp,)
    out = np.zeros((len(mon.omega_dt), len(comps), j1 - j0, i1 - i0), dtype=complex)
    for q, c in enumerate(comps):
        for n in range(n0, N + 1):
            x = hist[n - 1][c][k, j0:j1, i0:i1]
            if mon.kind == "flux_z" and c >= 3:
                below = hist[n - 1][c][k - 1, j0:j1, i0:i1] if k else np.zeros_like(x)
                x = dtype(0.5) * (x + below)
            for f, w in enumerate(mon.omega_dt):
                out[f, q] += x.astype(float) * np.exp(-1j * w * (n + (0.5 if c >= 3 else 0.0)))
    return out


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nf,chunk", [(1, 0), (3, 4), (4, 0), (5, 3), (9, 0)])
def test_spectra_of_all_monitors(dtype, nf, chunk):
    specs = [_spec(nf) for _ in range(4)]   # 20 monitors
    ref = Simulation(specs, dtype=dtype, max_steps=N)
    hist = []
    for d in range(4):
        _fill(ref, d)
    for _ in range(N):
        ref.step(1, record=False)
        hist.append([[ref.field(c, d) for c in range(6)] for d in range(4)])
    ref.close()
    sim = Simulation(specs, dtype=dtype, max_steps=N, dft_block=4, graph_chunk=chunk)
    for d in range(4):
        _fill(sim, d)
    if chunk:
        sim.step(N)
    else:   # monitor 1 of domain 2 starts over after step 3, one is read after step 6
        sim.step(3)
        sim.reset_monitor(1, 2)
        sim.step(3)
        sim.spectra(2, 1)
        sim.step(N - 6)
    for d in range(4):
        for m in range(5):
            n0 = 4 if not chunk and (d, m) == (2, 1) else 1
            want = _sum(specs[d], [h[d] for h in hist], m, n0, sim.dtype)
            # N terms below 6 (a few random states), each a product and a sum, and the factors' own rounding
            assert np.abs(sim.spectra(m, d) - want).max() <= 6.0 * N * (2 * N + 8) * 2.0 ** -53
    sim.close()

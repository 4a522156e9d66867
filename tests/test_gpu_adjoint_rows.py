"""The reverse field passes' branches: tile shapes, slot classes and films.

The tape schedule's gradients against the plain schedule's (other kernels:
every map on its own, by slots) on the grids where the passes branch: 256 x 1
tiles with x slabs and partial wavefronts, slots whose edge coefficients come
from the 16-bit classes, two films whose reaches overlap (the general form of
the film-region kernel), a film whose reach meets a CPML slab (no merged pass),
and a film alone in the box.  Both run in float64; the bound is the rounding of
a run of this length, as between the schedules elsewhere.
"""
import numpy as np
import pytest

from paper_2510_22221_amd import mpx
from synth import workloads as W

pytestmark = pytest.mark.gpu
N, N0 = 30, 12


def base(seed, n, bc, npml):
    w = W.random_case(seed, nx=n[0], ny=n[1], nz=n[2], bc=bc, npml=npml, film=False, nsteps=N)
    w.H0 = (3e6, 0.0, 5e6)
    return w


def wide():
    w = W.random_case(41, nx=520, ny=12, nz=10, bc=(W.PML, W.PML, W.PEC, W.PEC, W.PEC, W.PEC),
                      npml=(2, 2, 0, 0, 0, 0), nsteps=N)
    w.H0 = (3e6, 0.0, 5e6)
    return w


def classes():
    w = base(8, (40, 17, 13), (W.PML,) * 6, (3,) * 6)
    rng = np.random.default_rng(8)
    mats = [(float(rng.uniform(1.0, 12.0)), float(rng.uniform(0.0, 5e3)), 0, 0.0, 0.0, 0.0) for _ in range(150)]
    mats[3] = W.FILM
    mats[7] = W.PEC_METAL
    ids = rng.integers(4, 150, size=w.ids.shape).astype(np.uint8)
    ids[5:7, 6:11, 8:30] = 3
    w.materials, w.ids = mats, ids
    return w


def two_films():
    w = base(5, (34, 15, 12), (W.PEC,) * 6, (0,) * 6)
    w.ids[4:6, 5:10, 4:14] = 3
    w.ids[4:6, 5:10, 16:28] = 3
    return w


def near_slab():
    w = base(6, (31, 16, 14), (W.PML,) * 6, (3,) * 6)
    w.ids[5:7, 6:10, 12:27] = 3  # one cell before the slab at 28
    return w


def alone():
    w = base(7, (31, 16, 14), (W.PML,) * 6, (3,) * 6)
    w.ids[6:8, 6:10, 9:21] = 3
    return w


@pytest.mark.parametrize("case", [wide, classes, two_films, near_slab, alone])
def test_field_passes_match_plain_schedule(case):
    w = case()
    fc = np.argwhere(w.ids == 3)
    lo, hi = fc.min(axis=0), fc.max(axis=0)  # (k, j, i)
    eps_box = (int(lo[2]) - 2, int(lo[1]) - 1, int(lo[0]) - 2, 7, 4, 3)
    ms_box = tuple(int(v) for v in (lo[2], lo[1], lo[0], hi[2] - lo[2] + 1, hi[1] - lo[1] + 1, hi[0] - lo[0] + 1))
    out = []
    for sched in (0, 1):
        print(f"{case.__name__}: schedule {sched}", flush=True)
        g = mpx.from_workload(w, precision=mpx.F64)
        g.set_adjoint_schedule(sched)
        out.append(g.adjoint(N, N0, film=0, checkpoint_every=7, eps_box=eps_box, ms_box=ms_box))
        g.close()
    a, b = out
    assert a["loss"] == pytest.approx(b["loss"], rel=1e-13)
    for key in ("dH0", "deps", "dMs"):
        sc = float(np.abs(b[key]).max())
        assert sc > 0, key
        assert float(np.abs(a[key] - b[key]).max()) <= 1e-10 * sc, key

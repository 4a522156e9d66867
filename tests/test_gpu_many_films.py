"""Grids with as many films as a handle takes (64): the H/M pass finds the
films that meet a wavefront's row first, then their faces.

Against the fused sweep (which looks a face up in the film list by itself),
bitwise: films that start and end at, before and after a wavefront's and a
lane pair's bounds, thin ones, rows that meet several films.  And a step's time
must not grow with every film of the list.
"""
import time

import numpy as np
import pytest

from paper_2510_22221_amd import mpx
from synth import workloads as W

pytestmark = pytest.mark.gpu
PER, PEC, PML = W.PERIODIC, W.PEC, W.PML


def films(n, bc, npml, starts, widths, ny, nz):
    w = W.random_case(23, nx=n[0], ny=n[1], nz=n[2], bc=bc, npml=npml, film=False, nsteps=8)
    q = 0
    for k in range(nz):
        for j in range(ny):
            for i, m in zip(starts, widths):
                w.ids[4 + 5 * k:6 + 5 * k, 4 + 5 * j:7 + 5 * j, i:i + m] = 3 if q % 3 else 5
                q += 1
    w.H0 = (3e6, 0.0, 5e6)
    w.probes = []
    return w, q


CASES = [  # grid, boundaries, the films' x starts and widths, films along y and z
    ((135, 25, 16), (PEC,) * 6, (0,) * 6, (1, 5, 20, 40, 63, 66, 100, 126), (2, 10, 1, 20, 1, 31, 24, 4), 4, 2),
    ((200, 25, 16), (PML, PML, PEC, PEC, PEC, PEC), (3, 2, 0, 0, 0, 0), (5, 61, 65, 127, 131, 188), (54, 2, 60, 2, 50, 5), 4, 2),
    ((66, 25, 16), (PER, PER, PER, PER, PEC, PEC), (0,) * 6, (0,), (66,), 4, 2),
    ((530, 25, 16), (PEC,) * 6, (0,) * 6, (1, 255, 258, 300, 384, 400, 460, 515), (252, 1, 30, 70, 12, 50, 53, 13), 4, 2)]


@pytest.mark.parametrize("prec", [mpx.F64, mpx.F32])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_many_films_bitwise(case, prec):
    w, n = films(*CASES[case])
    out = []
    for schedule in (0, 1):
        print(f"case {case}, {n} films, prec={prec}, schedule={schedule}", flush=True)
        s = mpx.from_workload(w, precision=prec, graph_steps=2)
        s.set_schedule(schedule)
        assert s.info()["films"] == n
        rng = np.random.default_rng(case)
        for f in range(6):
            s.set(f, rng.standard_normal(s.get(f).shape) * (1.0 if f < 3 else 3e-3))
        for c in (1, 5):
            s.step(c)
        s.sync()
        out.append([s.get(f).copy() for f in range(12)])
        s.close()
    for f, (a, b) in enumerate(zip(*out)):
        assert np.isfinite(a).all() and np.any(a != 0.0) and np.array_equal(a, b), (case, f)


# (the films' own work aside: with every film looked at by every face, the step
# took 2.9 times as long with 48 small films as with one)
@pytest.mark.parametrize("prec", [mpx.F64, mpx.F32])
def test_step_time_does_not_grow_with_the_film_list(prec):
    best = []
    for count in (1, 48):
        w = W.box(200, 160, 40, bc=(PML,) * 6, npml=(4,) * 6)
        w.materials, w.H0 = list(W.BASE_TABLE), (0.0, 0.0, 8e4)
        for q in range(count):
            i, j = 10 + 22 * (q // 6), 10 + 24 * (q % 6)
            w.ids[20:24, j:j + 20, i:i + 18] = 3
        s = mpx.from_workload(w, precision=prec, graph_steps=64)
        s.step(128)
        s.sync()
        t = []
        for _ in range(6):
            t0 = time.perf_counter()
            s.step(128)
            s.sync()
            t.append(time.perf_counter() - t0)
        best.append(min(t) / 128 * 1e6)
        s.close()
    print(f"prec={prec}: one film {best[0]:.1f} us a step, 48 {best[1]:.1f}", flush=True)
    assert best[1] <= 2.2 * best[0]

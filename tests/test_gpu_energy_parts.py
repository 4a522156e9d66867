"""The energy sums over more partials than a launch has blocks (2048): the
blocks then loop.

A 301 x 141 x 13 grid has 2156 partials in the probe launch and 2340 tiles in
mpx_energy; a film of 400 x 140 x 10 cells has 2188 partials.  Both against the
same sums in numpy (and the oracle's energy) over the fields read back: every
term is of the sum's own sign or some three times it, and 3 10^6 of them in trees
of 256 round to some 10^-15 of it, well inside the bounds.
"""
import math

import numpy as np
import pytest

import oracle.oracle as O
from paper_2510_22221_amd import mpx
from synth import workloads as W

pytestmark = pytest.mark.gpu
MU0 = 4.0e-7 * math.pi
EPS0 = 1.0 / (MU0 * W.C0 ** 2)


def randomise(s, seed):
    rng = np.random.default_rng(seed)
    for f in range(6):
        s.set(f, rng.standard_normal(s.get(f).shape) * (1.0 if f < 3 else 3e-3))


@pytest.mark.parametrize("prec", [mpx.F64, mpx.F32])
@pytest.mark.parametrize("with_h", [False, True])
def test_grid_energy_of_looping_blocks(prec, with_h):
    w = W.random_case(9, nx=301, ny=141, nz=13, bc=(W.PERIODIC, W.PERIODIC, W.PEC, W.PEC, W.PEC, W.PEC), nsteps=3)
    w.probes = []
    print(f"301 x 141 x 13, prec={prec}, H probe={with_h}", flush=True)
    s = mpx.from_workload(w, precision=prec)
    pid = s.add_probe(mpx.PROBE_EM_ENERGY, cap=8)
    if with_h:
        s.add_probe(mpx.PROBE_FIELD, field=4, ijk=(7, 5, 4), cap=8)
    randomise(s, 4)
    s.step(3)
    got, probe = s.energy(), s.read_probe(pid, 1).ravel()[-1]
    o = O.from_workload(w)
    for f in range(6):
        o.set(f, s.get(f))
    for f in (6, 7, 8):
        o.set(f, s.get(f))
    ref = o.energy()
    print(f"  mpx_energy {got}, probe {probe}, oracle {ref}", flush=True)
    assert got[0] == pytest.approx(ref[0], rel=1e-12)
    assert got[1] == pytest.approx(ref[1], rel=1e-12)
    assert probe == pytest.approx(ref[0], rel=1e-12)
    assert s.energy()[0] == got[0]
    s.close()


# 5 x 5 x 4 cells: one partial; 2188; the most the H/M launch takes, and one more
@pytest.mark.parametrize("size", [(5, 5, 4), (400, 140, 10), (512, 128, 8), (512, 129, 8)])
def test_film_energy_of_looping_blocks(size):
    ni, nj, nk = size
    w = W.box(ni + 9, nj + 6, nk + 5, nsteps=2)
    w.materials = list(W.BASE_TABLE) + [(2.5, 0.0, 0, 0.9e5, 0.003, 1.9e11)]
    w.ids[2:2 + nk, 3:3 + nj, 4:4 + ni] = 3
    w.ids[2:4, 3:3 + nj // 2, 4:4 + ni // 2] = 4
    w.H0 = (3e6, 0.0, 5e6)
    print(f"film {size}: {-(-ni * nj * nk // 256)} partials", flush=True)
    s = mpx.from_workload(w, precision=mpx.F64)
    pid = s.add_probe(mpx.PROBE_FILM_ENERGY, film=0, cap=4)
    randomise(s, 5)
    s.step(2)
    got = s.read_probe(pid, 1).ravel()[-1]
    eps = np.zeros(w.ids.shape)
    mag = np.isin(w.ids, (3, 4))
    for q in (3, 4):
        eps[w.ids == q] = w.materials[q][0]
    we = np.zeros(w.ids.shape)
    wh = np.zeros(w.ids.shape)
    nz, ny, nx = w.ids.shape
    for c in range(3):  # natural dims [k, j, i]; axis a of the grid is axis 2 - a
        e2 = s.get(c) ** 2
        for a in range(3):
            if a != c:
                ax = 2 - a
                e2 = np.take(e2, range(0, w.ids.shape[ax]), ax) + np.take(e2, range(1, w.ids.shape[ax] + 1), ax)
        we += e2 / 4.0
        h2 = s.get(3 + c) ** 2
        ax = 2 - c
        wh += (np.take(h2, range(0, w.ids.shape[ax]), ax) + np.take(h2, range(1, w.ids.shape[ax] + 1), ax)) / 2.0
    ref = float((0.5 * EPS0 * eps * we + 0.5 * MU0 * wh)[mag].sum()) * math.prod(w.d)
    print(f"  probe {got}, numpy {ref}", flush=True)
    assert ref > 0.0 and got == pytest.approx(ref, rel=1e-12)
    s.close()

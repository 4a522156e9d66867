"""Grids on 64 x 4 tiles: the film's part of the H/M pass and the probes that
read only E, mean M or a film's energy ride in the H/M launch, alone and (E and
mean M) in batches.

One H-point probe more sends a simulation's probes to the probe launch; the
fields, the shared traces and the step counter must be the same bits.  The
cases differ in films (the probe block then follows no film block), in grid
size (the film and probe blocks fill part of a plane of tiles, or several) and
in the length of the calls (single steps run the bracket half steps only).
"""
import numpy as np
import pytest

from paper_2510_22221_amd import mpx
from synth import workloads as W

pytestmark = pytest.mark.gpu
CALLS = (1, 7, 1, 12, 5)


def case(film, n, seed):
    w = W.random_case(seed, nx=n[0], ny=n[1], nz=n[2], bc=(W.PML, W.PML, W.PEC, W.PEC, W.PEC, W.PEC),
                      npml=(2, 2, 0, 0, 0, 0), film=film, nsteps=sum(CALLS))
    w.H0 = (3e6, 0.0, 5e6)
    w.probes = []
    return w


def build(w, prec, film, with_h):
    s = mpx.from_workload(w, precision=prec, graph_steps=4)
    pids = [(s.add_probe(mpx.PROBE_FIELD, field=1, ijk=(6, 5, 4), cap=64), 1),
            (s.add_probe(mpx.PROBE_FIELD, field=2, ijk=(5, 4, 3), cap=64, every=3), 1)]
    if film:
        pids += [(s.add_probe(mpx.PROBE_MEAN_M, film=0, cap=64), 3),
                 (s.add_probe(mpx.PROBE_MEAN_M, film=0, cap=64, every=4), 3),
                 (s.add_probe(mpx.PROBE_FILM_ENERGY, film=0, cap=64), 1)]
    if with_h:
        s.add_probe(mpx.PROBE_FIELD, field=4, ijk=(7, 5, 4), cap=64)
    return s, pids


def state(s, pids):
    return [s.get(f).copy() for f in range(12)] + [s.read_probe(p, nv).copy() for p, nv in pids] + \
        [np.array(s.info()["step"])]


def same(a, b, what):
    assert len(a) == len(b)
    for q, (x, y) in enumerate(zip(a, b)):
        assert x.shape == y.shape and np.array_equal(x, y), (what, q)


@pytest.mark.parametrize("prec", [mpx.F64, mpx.F32])
@pytest.mark.parametrize("film,n", [(True, (23, 13, 11)), (True, (70, 29, 9)), (False, (23, 13, 11))])
def test_folded_probes_and_film_bitwise(prec, film, n):
    w = case(film, n, 7)
    out = []
    for with_h in (False, True):
        print(f"{n}, film={film}, H probe={with_h}, prec={prec}", flush=True)
        s, pids = build(w, prec, film, with_h)
        for c in CALLS:
            s.step(c)
        s.sync()
        out.append(state(s, pids))
        s.close()
    same(out[0], out[1], n)
    assert int(out[0][-1]) == sum(CALLS)
    assert all(np.any(t != 0.0) for t in out[0][12:-1])


@pytest.mark.parametrize("prec", [mpx.F64, mpx.F32])
def test_batch_of_folded_and_unfolded_members_bitwise(prec):
    spec = [(True, (23, 13, 11), False), (False, (31, 12, 10), False), (True, (40, 17, 9), True),
            (False, (19, 11, 9), True)]
    ws = [case(film, n, 7 + q) for q, (film, n, _) in enumerate(spec)]
    ref = []
    for w, (film, n, with_h) in zip(ws, spec):
        s, pids = build(w, prec, film, with_h)
        for c in CALLS:
            s.step(c)
        s.sync()
        ref.append(state(s, pids))
        s.close()
    members = [build(w, prec, film, with_h) for w, (film, n, with_h) in zip(ws, spec)]
    b = mpx.Batch([m[0] for m in members])
    b.set_graph_steps(4)
    for c in CALLS:
        b.step(c)
    b.sync()
    for q, (s, pids) in enumerate(members):
        print(f"member {q}, prec={prec}", flush=True)
        same(state(s, pids), ref[q], q)
    b.close()
    for s, _ in members:
        s.close()


@pytest.mark.parametrize("prec", [mpx.F64, mpx.F32])
@pytest.mark.parametrize("n", [(23, 13, 11), (301, 141, 13)])
def test_grid_energy_beside_the_hm_pass_bitwise(prec, n):
    # 13 partials, and 2156 (more than a launch has blocks for)
    w = W.random_case(9, nx=n[0], ny=n[1], nz=n[2], bc=(W.PERIODIC, W.PERIODIC, W.PEC, W.PEC, W.PEC, W.PEC),
                      film=True, nsteps=sum(CALLS))
    w.probes = []
    out = []
    for with_h in (False, True):
        print(f"{n}, H probe={with_h}, prec={prec}", flush=True)
        s = mpx.from_workload(w, precision=prec, graph_steps=4)
        pids = [(s.add_probe(mpx.PROBE_EM_ENERGY, cap=64), 1), (s.add_probe(mpx.PROBE_EM_ENERGY, cap=64, every=3), 1)]
        if with_h:
            s.add_probe(mpx.PROBE_FIELD, field=4, ijk=(7, 5, 4), cap=64)
        for c in CALLS:
            s.step(c)
        s.sync()
        out.append(state(s, pids))
        s.close()
    same(out[0], out[1], n)
    t, t3 = out[0][12], out[0][13]
    assert np.all(t > 0.0) and np.array_equal(t[2::3], t3)

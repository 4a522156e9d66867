"""Where a simulation's probes are sampled: in the H/M launch (one block, one
probe after another) while that costs less than the probe launch (a block a
probe), else there.

One H-point probe more sends every probe to the probe launch.  On both sides
of the line the fields, traces and step counter must be the same bits, and a
simulation with many probes must not be slower than with that one more.
"""
import time

import numpy as np
import pytest

from paper_2510_22221_amd import mpx
from synth import workloads as W

pytestmark = pytest.mark.gpu
CALLS = (1, 7, 4)
N = (24, 14, 12)


def build(n, prec, mix, with_h, cap=64):
    w = W.random_case(13, nx=n[0], ny=n[1], nz=n[2], nsteps=sum(CALLS))
    w.H0 = (3e6, 0.0, 5e6)
    w.probes = []
    s = mpx.from_workload(w, precision=prec, graph_steps=4)
    pids = []
    for q, ch in enumerate(mix):
        every = 1 + q % 3
        if ch == "E":
            pids.append((s.add_probe(mpx.PROBE_FIELD, field=q % 3, ijk=(5 + q % 8, 5, 4), cap=cap, every=every), 1))
        elif ch == "M":
            pids.append((s.add_probe(mpx.PROBE_MEAN_M, film=0, cap=cap, every=every), 3))
        else:
            kind = mpx.PROBE_FILM_ENERGY if ch == "F" else mpx.PROBE_EM_ENERGY
            pids.append((s.add_probe(kind, film=0, cap=cap, every=every), 1))
    if with_h:
        s.add_probe(mpx.PROBE_FIELD, field=4, ijk=(7, 5, 4), cap=cap)
    return s, pids


# few enough for the H/M launch, and one more than that
@pytest.mark.parametrize("prec", [mpx.F64, mpx.F32])
@pytest.mark.parametrize("mix", ["EEEE", "EEEEE", "MMM", "MMMM", "EEMM", "EEMMM", "FFF", "FFFF", "MF", "GG", "EMFG",
                                 "E" * 63])
def test_both_launches_bitwise(mix, prec):
    out = []
    for with_h in (False, True):
        print(f"{mix}, H probe={with_h}, prec={prec}", flush=True)
        s, pids = build(N, prec, mix, with_h)
        for c in CALLS:
            s.step(c)
        s.sync()
        out.append([s.get(f).copy() for f in range(12)] + [s.read_probe(p, nv).copy() for p, nv in pids]
                   + [np.array(s.info()["step"])])
        s.close()
    for q, (a, b) in enumerate(zip(*out)):
        assert a.shape == b.shape and np.array_equal(a, b), (mix, q)
    assert int(out[0][-1]) == sum(CALLS)
    assert all(np.any(t != 0.0) for t in out[0][12:-1])


# one after another in one block they took 3 to 7 times the step
@pytest.mark.parametrize("mix", ["E" * 63, "M" * 63])
def test_many_probes_do_not_wait_for_each_other(mix):
    best = []
    for with_h in (False, True):
        s, _ = build((64, 48, 40), mpx.F32, mix, with_h, cap=4096)
        s.set_graph_steps(64)
        s.step(256)
        s.sync()
        t = []
        for _ in range(7):
            t0 = time.perf_counter()
            s.step(256)
            s.sync()
            t.append(time.perf_counter() - t0)
        best.append(min(t) / 256 * 1e6)
        s.close()
    print(f"{mix[0]} x {len(mix)}: {best[0]:.1f} us a step, {best[1]:.1f} with an H probe more", flush=True)
    assert best[0] <= 1.3 * best[1]

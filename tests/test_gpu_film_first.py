"""The film's first half step with its prepass in one launch (up to 1024
blocks of 256 faces in a launch) and in two (above): the same bits.

A small film alone takes one launch; as a member of a batch beside a film of
more than 1024 blocks it takes two, and so does that one alone.  Films inside
walls, across one periodic axis and two, films of mixed materials, two films,
odd sizes; single steps (the bracket half steps) and runs of them.
"""
import numpy as np
import pytest

from paper_2510_22221_amd import mpx
from synth import workloads as W

pytestmark = pytest.mark.gpu
CALLS = (1, 6, 3)
PER, PEC = W.PERIODIC, W.PEC


def members():
    out = []
    for q, (n, bc) in enumerate([((23, 13, 11), (PEC,) * 6),
                                 ((21, 15, 12), (PER, PER, PEC, PEC, PEC, PEC)),
                                 ((17, 14, 12), (PER,) * 4 + (PEC, PEC)),
                                 ((26, 19, 17), (PEC,) * 6)]):
        w = W.random_case(11 + q, nx=n[0], ny=n[1], nz=n[2], bc=bc, film=q == 0, nsteps=sum(CALLS))
        if q == 1:
            w.ids[4:7, 4:9, :] = 3
        elif q == 2:
            w.ids[5:7] = 3
            w.ids[5, 3:6, 0:4] = 5
        elif q == 3:
            w.ids[2:5, 3:8, 4:20] = 3
            w.ids[9:14, 11:16, 5:9] = 5
        out.append(w)
    big = W.random_case(31, nx=400, ny=72, nz=9, film=False, nsteps=sum(CALLS))
    big.ids[2:6, 4:68, 10:390] = 3  # 381 x 65 x 5 faces a family: 1452 blocks
    out.append(big)
    for q, w in enumerate(out):
        w.probes = []
        w.H0 = (3e6, 0.0, 5e6)
        w.seed = q
    return out


def build(w, prec):
    s = mpx.from_workload(w, precision=prec, graph_steps=2)
    rng = np.random.default_rng(w.seed)
    for f in range(6):
        s.set(f, rng.standard_normal(s.get(f).shape) * (1.0 if f < 3 else 3e-3))
    nfilm = 2 if w.ids.shape == (17, 19, 26) else 1
    return s, [s.add_probe(mpx.PROBE_MEAN_M, film=f, cap=64) for f in range(nfilm)]


def state(m):
    s, pids = m
    return [s.get(f).copy() for f in range(12)] + [s.read_probe(p, 3).copy() for p in pids]


@pytest.mark.parametrize("prec", [mpx.F64, mpx.F32])
def test_one_launch_and_two_bitwise(prec):
    ws = members()
    alone = []
    for q, w in enumerate(ws):
        print(f"alone {q}, prec={prec}", flush=True)
        m = build(w, prec)
        for c in CALLS:
            m[0].step(c)
        m[0].sync()
        alone.append(state(m))
        m[0].close()
    ms = [build(w, prec) for w in ws]
    b = mpx.Batch([m[0] for m in ms])
    b.set_graph_steps(2)
    print(f"batch, prec={prec}", flush=True)
    for c in CALLS:
        b.step(c)
    b.sync()
    for q, m in enumerate(ms):
        got = state(m)
        assert np.any(got[9] != 0.0) and np.isfinite(got[9]).all()
        for f, (x, y) in enumerate(zip(got, alone[q])):
            assert np.array_equal(x, y), (q, f)
    b.close()
    for m in ms:
        m[0].close()

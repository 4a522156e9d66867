"""The shapes of the separate passes: two slots a lane in float64, one or
several wavefronts a row, rows that end inside a lane's pair, a wavefront or a
block -- against one slot a lane on 64 x 4 tiles (schedule 6), bitwise.
"""
import numpy as np
import pytest

from paper_2510_22221_amd import mpx
from synth import workloads as W

pytestmark = pytest.mark.gpu
PER, PEC, PML = W.PERIODIC, W.PEC, W.PML
CALLS = (1, 5)


def build(w, prec, schedule, seed):
    s = mpx.from_workload(w, precision=prec, graph_steps=2)
    if schedule:
        s.set_schedule(schedule)
    rng = np.random.default_rng(seed)
    for f in range(6):
        s.set(f, rng.standard_normal(s.get(f).shape) * (1.0 if f < 3 else 3e-3))
    return s


@pytest.mark.parametrize("prec", [mpx.F64, mpx.F32])
@pytest.mark.parametrize("nx", [64, 65, 97, 127, 128, 130, 191, 251, 513, 640, 1027])
def test_shapes_bitwise(prec, nx):
    ny, nz = (10, 9) if nx > 300 else (14, 9)
    for q, (bc, npml, uniform) in enumerate([((PEC,) * 6, (0,) * 6, False),
                                             ((PER,) * 6, (0,) * 6, False),
                                             ((PML, PML, PML, PEC, PEC, PML), (3, 2, 2, 0, 0, 2), False),
                                             ((PML, PML, PER, PER, PEC, PEC), (2, 5, 0, 0, 0, 0), True)]):
        w = W.random_case(50 + q, nx=nx, ny=ny, nz=nz, bc=bc, npml=npml, film=False, nsteps=sum(CALLS))
        if uniform:  # whole wavefronts of one class beside mixed ones
            w.ids[:, :, :] = 1
            w.ids[:, ny // 2:, nx // 2:] = 4
        w.ids[nz // 2:nz // 2 + 2, 4:ny - 4, max(12, nx // 2 - 20):nx // 2 + 20] = 3
        w.H0, w.probes = (3e6, 0.0, 5e6), []
        out = []
        for schedule in (0, 6):
            print(f"nx={nx}, prec={prec}, case {q}, schedule={schedule}", flush=True)
            s = build(w, prec, schedule, q)
            for c in CALLS:
                s.step(c)
            s.sync()
            out.append([s.get(f).copy() for f in range(12)])
            s.close()
        for f, (a, b) in enumerate(zip(*out)):
            assert np.isfinite(a).all() and np.array_equal(a, b), (q, f)
        assert all(np.any(a != 0.0) for a in out[0][:6])

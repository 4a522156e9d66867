"""Gradients with respect to the permittivity of boxes that do not align with
the lanes' pairs of slots: where the E pass holds two float64 slots a lane and
writes the box's tape, odd widths and starts, a box of one cell, one at a row's
end, one that reaches the periodic wrap.

The tape schedule (0) against the plain schedule (1), which forms every map by
slots; both float64, the bound the rounding of a run of this length, as between
the schedules elsewhere.
"""
import numpy as np
import pytest

from paper_2510_22221_amd import mpx
from synth import workloads as W

pytestmark = pytest.mark.gpu
N, N0 = 14, 5
PER, PEC, PML = W.PERIODIC, W.PEC, W.PML


@pytest.mark.parametrize("nx,bc,npml", [(128, (PML,) * 6, (3,) * 6), (127, (PER, PER, PER, PER, PEC, PEC), (0,) * 6),
                                        (251, (PEC,) * 6, (0,) * 6), (513, (PML, PML, PEC, PEC, PEC, PEC),
                                                                      (2, 2, 0, 0, 0, 0))])
@pytest.mark.parametrize("place", ["odd", "cell", "end"])
def test_tape_of_odd_boxes(nx, bc, npml, place):
    w = W.random_case(17, nx=nx, ny=14, nz=13, bc=bc, npml=npml, film=False, nsteps=N)
    edge = nx - npml[1]
    # a film whose waves reach the box and come back within the run
    i0 = edge - 20 if place == "end" else nx // 2 - 7
    w.ids[5:7, 5:9, i0:i0 + 13] = 3
    w.H0 = (3e6, 0.0, 5e6)
    box = {"odd": (nx // 2 - 9 | 1, 4, 4, 13, 5, 4), "cell": (nx // 2 + 7, 6, 6, 1, 1, 1),
           "end": (edge - 5, 3, 3, 5, 3, 3)}[place]
    # a current beside the box: every place's gradient is above rounding
    w.sources = [W.Source(2, (box[0] - 2, box[1], box[2], 2, 2, 1), 1e9 * np.sin(0.3 * np.arange(N) + 0.5))]
    out = []
    for sched in (0, 1):
        print(f"nx={nx}, box {box}, schedule {sched}", flush=True)
        s = mpx.from_workload(w, precision=mpx.F64)
        rng = np.random.default_rng(3)
        for f in range(6):
            s.set(f, rng.standard_normal(s.get(f).shape) * (1.0 if f < 3 else 3e-3))
        s.set_adjoint_schedule(sched)
        out.append(s.adjoint(N, N0, film=0, checkpoint_every=5, eps_box=box))
        s.close()
    a, b = out
    assert a["loss"] == pytest.approx(b["loss"], rel=1e-13)
    for key in ("dH0", "deps"):
        sc = float(np.abs(b[key]).max())
        assert sc > 0 and float(np.abs(a[key] - b[key]).max()) <= 1e-10 * sc, key

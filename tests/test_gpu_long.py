"""A long narrow grid whose film fills most of its cross section: its film
blocks are more than a launch's z grid holds beside the planes of tiles, so
they take a launch of their own, before the tiles'.

Against the fused sweep (which launches the film's half steps by themselves,
one-dimensional), bitwise, with a probe block and without.
"""
import numpy as np
import pytest

from paper_2510_22221_amd import mpx
from synth import workloads as W

pytestmark = pytest.mark.gpu
NZ = 18600  # with 63 x 7 x (NZ - 3) faces a family: 18600 + 48052 planes


@pytest.mark.parametrize("probes", [False, True])
def test_film_blocks_past_the_z_grid(probes):
    w = W.box(64, 8, NZ, nsteps=4)
    w.materials = list(W.BASE_TABLE)
    w.ids[:, :3] = 1
    w.ids[2:NZ - 2, 1:7, 1:63] = 3
    w.H0 = (3e6, 0.0, 5e6)
    w.sources = [W.Source(2, (5, 3, 2, 40, 2, NZ - 5), 1e9 * np.sin(0.4 * np.arange(4) + 0.3))]
    blocks = 3 * -(-63 * 7 * (NZ - 3) // 256)
    assert NZ + blocks // 2 > 65536 and NZ < 65536
    boxes = [(0, 0, 0, 64, 8, 12), (0, 0, NZ // 2, 64, 8, 12), (0, 0, NZ - 12, 64, 8, 12)]
    out = []
    for schedule in (0, 1):
        print(f"64 x 8 x {NZ}, schedule {schedule}, probes={probes}", flush=True)
        s = mpx.from_workload(w, precision=mpx.F32, graph_steps=2)
        s.set_schedule(schedule)
        if probes:
            p = s.add_probe(mpx.PROBE_FIELD, field=2, ijk=(20, 3, NZ - 10), cap=16)
        for c in (1, 3):
            s.step(c)
        s.sync()
        got = [s.get_region(f, b) for f in (0, 2, 3, 4, 9, 11) for b in boxes] + [np.array(s.info()["step"])]
        if probes:
            got.append(s.read_probe(p, 1))
        out.append(got)
        s.close()
    for q, (a, b) in enumerate(zip(*out)):
        assert np.any(a != 0.0) and np.array_equal(a, b), q

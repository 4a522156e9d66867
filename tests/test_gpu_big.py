"""Arrays of 4 GiB and more: the passes then address a plane at a time.

What happens near the high corner of such a grid is what happens near that of
a small one as wide: fields that start in a window at the corner, with random
media, a film and CPML slabs, have not left it after a few steps, so the
window must hold the same bits.  Stepping alone, as a member of a batch beside
a small one (the batch then runs the large form for both), and the gradients
of a weighted trace (float64), whose E pass writes the tape.
"""
import numpy as np
import pytest
import torch

from paper_2510_22221_amd import mpx
from synth import workloads as W

pytestmark = pytest.mark.gpu
NX, WIN, EDGE = 600, 44, 16  # the window's rows and planes; the first of them that stay zero at the start
PML, PEC = W.PML, W.PEC
STEPS = (2, 1)


def window(many):
    """the small grid: its low y and z walls lie where the large one goes on
    (many: more distinct edge coefficients than the class byte holds)"""
    w = W.box(NX, WIN, WIN, d=(2e-6, 1.5e-6, 1e-6), bc=(PML, PML, PEC, PML, PEC, PML), npml=(4, 3, 0, 3, 0, 5),
              nsteps=12)
    rng = np.random.default_rng(77)
    w.materials = list(W.BASE_TABLE) + [(7.0, 2e3, 0, 0.0, 0.0, 0.0)]
    w.ids[EDGE:, EDGE:] = rng.choice([0, 1, 2, 4], p=[0.5, 0.3, 0.02, 0.18], size=(WIN - EDGE, WIN - EDGE, NX))
    if many:
        w.materials += [(float(v), 0.0, 0, 0.0, 0.0, 0.0) for v in rng.uniform(1.0, 12.0, size=60)]
        w.ids[30:, 30:] = rng.integers(4, 64, size=(WIN - 30, WIN - 30, NX))
    w.ids[22:24, 20:30, 200:400] = 0
    w.ids[24:26, 21:29, 210:390] = 3
    w.H0, w.m_dir = (3e6, 0.0, 5e6), (0.3, 0.1, 1.0)
    w.sources = [W.Source(2, (300, 30, 30, 4, 2, 2), 1e9 * np.sin(0.4 * np.arange(12) + 0.3))]
    return w


def large(w, ny, nz):
    """the same at the high corner of an NX x ny x nz grid"""
    b = W.Workload("large", NX, ny, nz, w.d, w.dt, w.courant, bc=w.bc, npml=w.npml, materials=w.materials,
                   ids=np.zeros((nz, ny, NX), dtype=np.uint8), H0=w.H0, m_dir=w.m_dir, nsteps=w.nsteps)
    b.ids[nz - WIN:, ny - WIN:] = w.ids
    for s in w.sources:
        i, j, k, ni, nj, nk = s.box
        b.sources.append(W.Source(s.comp, (i, j + ny - WIN, k + nz - WIN, ni, nj, nk), s.table))
    return b


def start(w, prec):
    s = mpx.from_workload(w, precision=prec, graph_steps=2)
    for f in range(6):
        g = torch.Generator().manual_seed(f)
        v = torch.randn((WIN, WIN, NX), generator=g, dtype=torch.float64) * (1.0 if f < 3 else 3e-3)
        v[:EDGE] = 0.0
        v[:, :EDGE] = 0.0
        if f < 3:  # conductor and wall edges hold no field
            pec = torch.as_tensor(w.ids[-WIN:, -WIN:] == 2)
            for a in range(3):
                if a != f:
                    pec = pec | pec.roll(1, 2 - a)
            v[pec] = 0.0
            if f != 0:
                v[:, :, 0] = 0.0
        s.storage(f)[-WIN:, -WIN:].copy_(v.to(s.storage(f).dtype))
    torch.cuda.synchronize()
    return s


def same(big, small, what):
    big.sync()
    small.sync()
    for f in range(6):
        a, b = big.storage(f)[-WIN:, -WIN:], small.storage(f)
        assert bool(torch.isfinite(b).all()) and bool((b != 0).any()), (what, f)
        assert torch.equal(a, b), (what, f)
        # nothing has come near the window's open sides
        assert not bool((b[:2] != 0).any()) and not bool((b[:, :2] != 0).any()), (what, f)
    nz, ny, _ = big.shape
    for c in range(3):
        box = (205, 18, 20, 190, 14, 8)
        a = big.get_region(9 + c, (box[0], box[1] + ny - WIN, box[2] + nz - WIN) + box[3:])
        b = small.get_region(9 + c, box)
        assert np.any(b != 0.0) and np.array_equal(a, b), (what, 9 + c)


@pytest.mark.parametrize("prec,ny,nz,many", [(mpx.F64, 890, 1010, False), (mpx.F64, 890, 1010, True),
                                             (mpx.F32, 1100, 1640, False), (mpx.F32, 1100, 1640, True)])
def test_high_corner_bitwise(prec, ny, nz, many):
    esz = 8 if prec == mpx.F64 else 4
    assert 608 * ny * (nz - 10) * esz > 2 ** 32
    w = window(many)
    print(f"600 x {ny} x {nz}, prec={prec}, many={many}: setup", flush=True)
    big = start(large(w, ny, nz), prec)
    small = start(w, prec)
    third = start(w, prec)  # the batch's small member, compared with one that steps alone
    alone = start(w, prec)
    print("  stepping", flush=True)
    for n in STEPS:
        big.step(n)
        small.step(n)
    same(big, small, "alone")
    print("  batch", flush=True)
    b = mpx.Batch([third, big])
    b.set_graph_steps(2)
    b.step(3)
    b.sync()
    small.step(3)
    same(big, small, "batch")
    alone.step(3)
    same(third, alone, "batch, small member")
    b.close()
    if prec == mpx.F64:
        print("  gradients", flush=True)
        out = []
        for s, (oy, oz) in ((big, (ny - WIN, nz - WIN)), (small, (0, 0))):
            out.append(s.adjoint_probe(3, 2, (301, 31 + oy, 31 + oz), [1.0, -0.7, 0.4], checkpoint_every=2,
                                       eps_box=(297, 28 + oy, 29 + oz, 7, 5, 4),
                                       ms_box=(205, 20 + oy, 23 + oz, 9, 10, 4)))
        same(big, small, "gradients")
        for key in ("dH0", "deps", "dMs"):
            assert np.array_equal(out[0][key], out[1][key]), key
        assert out[0]["loss"] == out[1]["loss"] and np.any(out[0]["deps"] != 0.0)
    for s in (big, small, third, alone):
        s.close()

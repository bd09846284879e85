"""The four-nodes-per-thread finite-difference update against the tile of one node per thread.

A forward that also returns energies runs the tile, one that does not the rows of quads, with the
same arithmetic in the same order: the traces are equal bit for bit, and so are the gradients of
the two z-chunks (the streaming variant is forced on small grids by DD_FD_NT=1).  Row lengths of every
remainder by four, planes that fill blocks in part and in full, single-plane remainders of both chunks, boxes at
the margin, all kinds of faces, dipoles in corners, one launch and two per step.
"""

import math

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

SIDES = synth.FACE_XMIN | synth.FACE_XMAX | synth.FACE_YMIN | synth.FACE_YMAX
TB = synth.FACE_TOP | synth.FACE_BOTTOM
FORMS = {
    # name: (n_outer, fem_lo, fem_cells, n_steps, detector faces, absorbing faces, ckpt_every, source)
    "minimal": ((5, 5, 5), (1, 1, 1), (2, 2, 2), 12, synth.FACE_ALL, TB | SIDES, 5, "plane"),
    "two_quads": ((6, 41, 7), (1, 3, 1), (3, 30, 4), 20, synth.FACE_XMAX | synth.FACE_TOP, TB, 7, "oblique"),
    "three_over": ((35, 33, 31), (9, 8, 7), (17, 16, 18), 40, SIDES, TB | SIDES, 8, "oblique"),
    "full_blocks": ((64, 64, 24), (15, 1, 5), (33, 61, 14), 30, synth.FACE_ALL, TB, 30, "corner"),
    "one_wave": ((32, 8, 40), (4, 1, 7), (25, 5, 26), 30, synth.FACE_YMIN | synth.FACE_BOTTOM, SIDES, 11, "edge"),
    "long_rows": ((261, 9, 13), (100, 2, 3), (31, 5, 7), 24, synth.FACE_TOP, 0, 6, "plane"),
    "many_blocks": ((70, 67, 65), (11, 20, 13), (41, 32, 44), 18, synth.FACE_TOP | synth.FACE_YMAX, TB, 6, "plane"),
}


@pytest.mark.parametrize("fused", ["1", "0"])
@pytest.mark.parametrize("name", sorted(FORMS))
def test_rows_equal_tiles_bit_for_bit(name, fused, monkeypatch):
    import torch
    from paper_2508_07780_amd import Problem
    n, lo, cells, nt, det, damp, ck, kind = FORMS[name]
    h = 0.05
    d = synth.ProblemDesc(n_outer=n, h=h, origin=(0.0, 0.0, 0.0), fem_lo=lo, fem_cells=cells,
                          dt=0.5 * h / math.sqrt(3.0), n_steps=nt, ckpt_every=ck, detector_faces=det,
                          absorbing_faces=damp)
    rng = np.random.Generator(np.random.PCG64(2508077800 + 950 + sorted(FORMS).index(name)))
    free = synth.fem_layers(d) >= 2
    eps = torch.tensor(np.where(free, 1.0 + 3.0 * rng.random(free.shape), 1.0), dtype=torch.float32, device="cuda")
    sig = torch.tensor(np.where(free, 0.8 * rng.random(free.shape), 0.0), dtype=torch.float32, device="cuda")
    base = synth.gauss_sine(2 * math.pi / (8 * h), pol=(0.3, 1.0, -0.4))
    d.t_switch = base.support_end() if kind != "corner" else 0.0
    dip = dict(kind=synth.SRC_DIPOLE, omega=base.omega, t0=base.t0, width=base.width, pol=(0.5, -0.2, 1.0))
    src = {"plane": lambda: base,
           "oblique": lambda: synth.Source(kind=base.kind, omega=base.omega, t0=base.t0, width=base.width,
                                           pol=(0.0, 1.0, 0.0), dir=(0.4, 0.0, -math.sqrt(1 - 0.16))),
           "corner": lambda: synth.Source(pos=(n[0] - 1, 0, n[2] - 1), **dip),
           "edge": lambda: synth.Source(pos=(n[0] - 1, n[1] // 2, 0), **dip)}[kind]()
    cot = None
    grads = []
    monkeypatch.setenv("DD_RESIDENT", "0")
    monkeypatch.setenv("DD_FUSED", fused)
    for stream in ("0", "1"):
        print(f"[gpu] {name} DD_FUSED={fused} DD_FD_NT={stream}", flush=True)
        monkeypatch.setenv("DD_FD_NT", stream)
        p = Problem(d)
        p.set_coefficients(eps, sig)
        tiles = p.forward([src], save=False, energy=True)[0].clone()
        rows = p.forward([src], save=True).clone()
        assert torch.isfinite(rows).all() and float(rows.abs().max()) > 0
        assert torch.equal(tiles.view(torch.int32), rows.view(torch.int32))
        if cot is None:
            cot = torch.tensor(rng.standard_normal(tuple(rows.shape)), dtype=torch.float32, device="cuda")
        p.adjoint(cot)
        grads.append([g.clone() for g in p.gradient()])
        p.adjoint_misfit(rows, 0.5 * cot)
        grads[-1] += [g.clone() for g in p.gradient()]
        torch.cuda.synchronize()
        p.close()
    for a, b in zip(*grads):
        assert torch.equal(a.view(torch.int64), b.view(torch.int64))

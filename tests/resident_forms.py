"""Problems that between them take every variant of the resident kernels."""

import math

import numpy as np

import synth

TB = synth.FACE_TOP | synth.FACE_BOTTOM
ALL = synth.FACE_ALL
TOP = synth.FACE_TOP
LONG = 100         # one checkpoint segment: the adjoint recomputes nothing
# name: (n_outer, fem_lo, fem_cells, detector faces, absorbing faces, ckpt_every, source,
#        forward (planes per thread, FEM nodes per thread), adjoint (the same))
VARIANTS = {
    "a4_rec": ((23, 29, 20), (5, 5, 11), (6, 9, 4), TOP, ALL, 5, "face", (2, 1), (4, 1)),
    "a2": ((57, 26, 28), (4, 14, 3), (15, 2, 23), TOP, TB, LONG, "plane", (2, 1), (2, 1)),
    "f4": ((61, 37, 42), (13, 1, 1), (46, 27, 39), TOP, ALL, 6, "corner", (4, 1), (8, 1)),
    "cube64": ((64, 64, 64), (16, 16, 16), (32, 32, 32), ALL, TB, LONG, "inside", (4, 1), (4, 1)),
    "cube64_rec": ((64, 64, 64), (16, 16, 16), (32, 32, 32), TOP, TB, 7, "oblique", (4, 1), (8, 1)),
    "f4_fem2": ((29, 110, 61), (3, 15, 2), (24, 86, 50), TOP, TB, LONG, "plane", (4, 2), (8, 2)),
    "cube96": ((96, 96, 96), (24, 24, 24), (48, 48, 48), TOP, TB, LONG, "face", (8, 3), (12, 2)),
    "cube96_rec": ((96, 96, 96), (24, 24, 24), (48, 48, 48), TOP, TB, 6, "plane", (8, 3), (12, 2)),
    "run9_dipole": ((100, 100, 100), (30, 30, 30), (40, 40, 40), TOP, TB, LONG, "inside", (12, 3), (12, 2)),
    "run12_rec": ((100, 100, 100), (30, 30, 30), (40, 40, 40), TOP, TB, 6, "corner", (12, 3), (12, 2)),
    "sides_rec": ((98, 43, 43), (2, 1, 1), (77, 37, 40), ALL, ALL, 6, "plane", (8, 2), (8, 2)),
    "f12_fem2": ((127, 96, 97), (96, 2, 52), (3, 84, 34), TOP, TB, LONG, "oblique", (12, 2), (12, 2)),
    "f12_fem3": ((67, 67, 90), (3, 7, 9), (55, 54, 78), ALL, TB, LONG, "plane", (12, 3), (8, 3)),
    "fem3_rec": ((37, 82, 119), (1, 21, 10), (33, 57, 107), TOP, TB, 6, "oblique", (8, 3), (12, 3)),
}
STEPS = 17


def variant(planes, nodes):
    """The kernel variant of a plan: planes per thread it holds, finite-element nodes per thread."""
    return (next(k for k in (2, 4, 8, 12) if planes <= k), (nodes + 511) // 512)


def problem(name):
    """(descriptor, eps, sigma, sources) of a variant's problem."""
    n, lo, cells, det, damp, ck, kind, _, _ = VARIANTS[name]
    h = 0.05
    d = synth.ProblemDesc(n_outer=n, h=h, origin=(0.0, 0.0, 0.0), fem_lo=lo, fem_cells=cells,
                          dt=0.5 * h / math.sqrt(3.0), n_steps=STEPS, ckpt_every=ck, detector_faces=det,
                          absorbing_faces=damp)
    rng = np.random.Generator(np.random.PCG64(2508077800 + 970 + sorted(VARIANTS).index(name)))
    free = synth.fem_layers(d) >= 2
    eps = np.where(free, 1.0 + 3.0 * rng.random(free.shape), 1.0)
    sig = np.where(free, 0.8 * rng.random(free.shape), 0.0)
    base = synth.gauss_sine(2 * math.pi / (8 * h), pol=(0.3, 1.0, -0.4))
    d.t_switch = base.support_end()
    dip = dict(kind=synth.SRC_DIPOLE, omega=base.omega, t0=base.t0, width=base.width, pol=(0.5, -0.2, 1.0))
    nx, ny, nz = n
    one = {"plane": lambda: base,
           "oblique": lambda: synth.Source(kind=base.kind, omega=base.omega, t0=base.t0, width=base.width,
                                           pol=(0.0, 1.0, 0.0), dir=(0.4, 0.0, -math.sqrt(1 - 0.16))),
           "corner": lambda: synth.Source(pos=(0, 0, 0), **dip),
           "face": lambda: synth.Source(pos=(nx - 1, ny // 2, nz // 2), **dip),
           "inside": lambda: synth.Source(pos=(nx // 2, 2, nz - 3), **dip)}[kind]()
    return d, eps, sig, [one, base]

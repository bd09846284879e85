"""Resident solves (all steps of a source in one launch) against solves by one launch per step.

Both orders of the arithmetic are the same, so everything a call returns is equal bit for bit:
traces, interface history through the gradients, and the fields' energies of the calls after it.

* bricks at the edges of their ranges: one brick, the smallest problem, single-node remainders in
  every axis, a FEM box against the margin, on brick boundaries, larger than half the grid, one to
  three nodes per thread of a FEM brick, runs of 1 to 12 planes, side detectors, absorbing sides,
  dipoles on faces and inside, oblique waves, one and several checkpoint segments;
* the one-block kernel that takes a solve whose blocks did not get their places;
* several problems on streams of their own, from threads;
* a solve whose first values are not finite;
* a caller's capture, which runs by launches, between resident solves.
"""

import math
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

SIDES = synth.FACE_XMIN | synth.FACE_XMAX | synth.FACE_YMIN | synth.FACE_YMAX
TB = synth.FACE_TOP | synth.FACE_BOTTOM
FORMS = {
    # name: (n_outer, fem_lo, fem_cells, n_steps, detector faces, absorbing faces, ckpt_every, source)
    "minimal": ((5, 5, 5), (1, 1, 1), (2, 2, 2), 6, synth.FACE_ALL, TB, 1, "plane"),
    "four_steps": ((12, 11, 13), (3, 3, 4), (5, 4, 5), 4, synth.FACE_ALL, TB, 3, "face"),
    "margin": ((14, 12, 16), (1, 1, 1), (11, 9, 13), 30, synth.FACE_BOTTOM, TB, 100, "corner"),
    "one_over": ((33, 33, 33), (8, 9, 7), (17, 16, 18), 40, synth.FACE_ALL, TB, 8, "plane"),
    "thin": ((65, 6, 20), (10, 1, 5), (33, 2, 9), 35, synth.FACE_YMIN, TB | SIDES, 8, "plane"),
    "flat": ((40, 41, 5), (3, 5, 1), (33, 31, 2), 30, synth.FACE_TOP, SIDES, 16, "corner"),
    "sides": ((36, 35, 34), (10, 3, 16), (16, 26, 16), 33, SIDES, TB | SIDES, 5, "oblique"),
    "no_damping": ((20, 37, 26), (4, 6, 7), (12, 24, 13), 33, synth.FACE_TOP, 0, 64, "inside"),
    "brick_edges": ((64, 32, 48), (16, 8, 16), (33, 17, 17), 24, synth.FACE_ALL, TB, 24, "face"),
    "mostly_fem": ((30, 31, 32), (2, 2, 2), (25, 26, 27), 24, synth.FACE_TOP, TB, 7, "plane"),
    "large": ((98, 93, 87), (20, 23, 18), (49, 41, 45), 17, synth.FACE_TOP | synth.FACE_XMAX, TB, 6, "oblique"),
    "wide_fd": ((101, 96, 94), (43, 40, 41), (11, 12, 9), 17, synth.FACE_TOP, TB, 32, "plane"),
}


def _form(name):
    n, lo, cells, nt, det, damp, ck, kind = FORMS[name]
    h = 0.05
    d = synth.ProblemDesc(n_outer=n, h=h, origin=(0.0, 0.0, 0.0), fem_lo=lo, fem_cells=cells,
                          dt=0.5 * h / math.sqrt(3.0), n_steps=nt, ckpt_every=ck, detector_faces=det,
                          absorbing_faces=damp)
    rng = np.random.Generator(np.random.PCG64(2508077800 + 900 + sorted(FORMS).index(name)))
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


def _problem(torch, monkeypatch, form, mode, allocator="torch"):
    from paper_2508_07780_amd import Problem
    monkeypatch.setenv("DD_RESIDENT", str(mode))
    d, eps, sig, _ = form
    p = Problem(d, allocator=allocator)
    p.set_coefficients(torch.tensor(eps, dtype=torch.float32, device="cuda"),
                       torch.tensor(sig, dtype=torch.float32, device="cuda"))
    return p


def _run(torch, p, sources, obs=None):
    """Two saved forwards and the gradients of a misfit and of a cotangent, then a forward without saving."""
    out = []
    for s in (sources, sources[::-1]):
        tr = p.forward(s, save=True).clone()
        p.adjoint_misfit(tr, 0.5 * tr if obs is None else obs)
        out += [tr] + [g.clone() for g in p.gradient()]
        p.adjoint((0.3 * tr).contiguous())
        out += [g.clone() for g in p.gradient()]
    out.append(p.forward(sources, save=False).clone())
    torch.cuda.synchronize()
    return out


def _same(torch, a, b):
    return [bool(torch.equal(x.view(torch.uint8), y.view(torch.uint8))) for x, y in zip(a, b)]


@pytest.mark.parametrize("name", sorted(FORMS))
def test_equals_launches_bit_for_bit(name, monkeypatch):
    import torch
    form = _form(name)
    got, held = [], []
    for mode in (0, 1):
        print(f"[gpu] {name} DD_RESIDENT={mode}", flush=True)
        p = _problem(torch, monkeypatch, form, mode)
        got.append(_run(torch, p, form[3]))
        held.append(p.device_bytes())
        assert torch.isfinite(got[-1][0]).all() and float(got[-1][0].abs().max()) > 0
        p.close()
    assert held[1] > held[0]                                   # the plans' lists and words: it did run resident
    assert all(_same(torch, *got)), _same(torch, *got)


@pytest.mark.parametrize("name", ["minimal", "four_steps", "thin", "sides", "no_damping"])
def test_one_block_kernel(name, monkeypatch):
    import torch
    form = _form(name)
    got = []
    for mode in (0, 2):
        print(f"[gpu] {name} DD_RESIDENT={mode}", flush=True)
        p = _problem(torch, monkeypatch, form, mode)
        got.append(_run(torch, p, form[3][:1]))
        p.close()
    assert all(_same(torch, *got)), _same(torch, *got)


def test_streams_and_threads(monkeypatch):
    import torch
    names = ["one_over", "sides", "large", "wide_fd", "one_over", "large"]
    forms = [_form(n) for n in names]
    want = []
    for f in forms:
        p = _problem(torch, monkeypatch, f, 0)
        want.append(_run(torch, p, f[3]))
        p.close()
    ps = [_problem(torch, monkeypatch, f, 1) for f in forms]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in forms]
    got, errors = [None] * len(forms), []

    def work(i):
        try:
            with torch.cuda.stream(streams[i]):
                for _ in range(3):
                    out = _run(torch, ps[i], forms[i][3])
                    assert all(_same(torch, out, want[i])), (names[i], _same(torch, out, want[i]))
                got[i] = out
        except BaseException as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(forms))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for p in ps:
        p.close()
    assert not errors, errors


def test_values_that_are_not_finite(monkeypatch):
    import torch
    form = _form("one_over")
    src = form[3][1]
    src.amp = 1.0e42                        # finite in 64 bits, infinite in 32
    got = []
    for mode in (0, 1):
        p = _problem(torch, monkeypatch, form, mode)
        tr = p.forward([src], save=True).clone()
        cot = torch.zeros_like(tr)
        cot[0, -3, 5, 1] = float("inf")
        p.adjoint(cot)
        got.append([tr.isnan(), tr.nan_to_num()] + [x for g in p.gradient() for x in (g.isnan(), g.nan_to_num())])
        torch.cuda.synchronize()
        p.close()
    assert not bool(torch.isfinite(tr).all())
    assert all(_same(torch, *got)), _same(torch, *got)


def test_between_captures_of_the_caller(monkeypatch):
    import torch
    form = _form("one_over")
    p = _problem(torch, monkeypatch, form, 1)
    tr = p.forward(form[3], save=True)
    want = tr.clone()
    out = torch.zeros_like(tr)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        p.forward(form[3], save=False, out=out)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert torch.equal(p.forward(form[3], out=tr), want)
    p.close()

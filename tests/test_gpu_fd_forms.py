"""The two forms of the finite-difference update, the tile of one node per thread and the rows of four, in every
kernel that has both: forced on the same problem by DD_FD_ROWS they give the same bits.

Problems of test_gpu_rows (row lengths of every remainder, single planes, all kinds of faces, dipoles, oblique
waves); one launch and two per step, the form R2, the paper-formula gradient, segments recomputed, batched jobs
alone and together.
"""

import math

import numpy as np
import pytest

import synth
from tests.test_gpu_rows import FORMS

pytestmark = pytest.mark.gpu


def _form(name):
    n, lo, cells, nt, det, damp, ck, kind = FORMS[name]
    h = 0.05
    d = synth.ProblemDesc(n_outer=n, h=h, origin=(0.0, 0.0, 0.0), fem_lo=lo, fem_cells=cells,
                          dt=0.5 * h / math.sqrt(3.0), n_steps=nt, ckpt_every=ck, detector_faces=det,
                          absorbing_faces=damp)
    rng = np.random.Generator(np.random.PCG64(2508077800 + 990 + sorted(FORMS).index(name)))
    free = synth.fem_layers(d) >= 2
    eps = np.where(free, 1.0 + 3.0 * rng.random(free.shape), 1.0).astype(np.float32)
    sig = np.where(free, 0.8 * rng.random(free.shape), 0.0).astype(np.float32)
    base = synth.gauss_sine(2 * math.pi / (8 * h), pol=(0.3, 1.0, -0.4))
    d.t_switch = base.support_end()
    dip = dict(kind=synth.SRC_DIPOLE, omega=base.omega, t0=base.t0, width=base.width, pol=(0.5, -0.2, 1.0))
    src = {"plane": lambda: base,
           "oblique": lambda: synth.Source(kind=base.kind, omega=base.omega, t0=base.t0, width=base.width,
                                           pol=(0.0, 1.0, 0.0), dir=(0.4, 0.0, -math.sqrt(1 - 0.16))),
           "corner": lambda: synth.Source(pos=(n[0] - 1, 0, n[2] - 1), **dip),
           "edge": lambda: synth.Source(pos=(n[0] - 1, n[1] // 2, 0), **dip)}[kind]()
    return d, eps, sig, src


def _problem(torch, form):
    from paper_2508_07780_amd import Problem
    p = Problem(form[0])
    p.set_coefficients(torch.tensor(form[1], device="cuda"), torch.tensor(form[2], device="cuda"))
    return p


def _bits(torch, x):
    return x.contiguous().view(torch.uint8)


@pytest.mark.parametrize("how", ["one_launch", "two_launches", "r2", "paper"])
@pytest.mark.parametrize("name", sorted(FORMS))
def test_forms_equal_bit_for_bit(name, how, monkeypatch):
    import torch
    form = _form(name)
    monkeypatch.setenv("DD_RESIDENT", "0")
    monkeypatch.setenv("DD_FUSED", "0" if how == "two_launches" else "1")
    got = []
    for rows in ("0", "1"):
        print(f"[gpu] {name} {how} DD_FD_ROWS={rows}", flush=True)
        monkeypatch.setenv("DD_FD_ROWS", rows)
        p = _problem(torch, form)
        if how == "r2":
            p.set_divdiv_form("R2")
        if how == "paper":
            p.paper_gradient(True)
        tr = p.forward([form[3]], save=True).clone()
        assert torch.isfinite(tr).all() and float(tr.abs().max()) > 0
        out = [tr]
        p.adjoint((0.3 * tr).contiguous())
        out += [g.clone() for g in p.gradient()]
        p.adjoint_misfit(tr, 0.5 * tr)
        out += [g.clone() for g in p.gradient()]
        torch.cuda.synchronize()
        p.close()
        got.append(out)
    for i, (a, b) in enumerate(zip(*got)):
        if how in ("r2", "paper") and i:       # their gradient terms add up by atomics, in any order
            assert float((a - b).norm()) <= 1e-12 * float(b.norm())
        else:
            assert torch.equal(_bits(torch, a), _bits(torch, b))


@pytest.mark.parametrize("names", [["three_over"], ["one_wave"], ["minimal", "full_blocks", "two_quads"]])
def test_batched_forms_equal_bit_for_bit(names, monkeypatch):
    import torch
    from paper_2508_07780_amd.batch import Batch
    forms = [_form(n) for n in names]
    got = []
    for rows in ("0", "1"):
        print(f"[gpu] batch {names} DD_FD_ROWS={rows}", flush=True)
        monkeypatch.setenv("DD_FD_ROWS", rows)
        ps = [_problem(torch, f) for f in forms]
        b = Batch(len(ps))
        ids = []
        for p, f in zip(ps, forms):
            obs = torch.linspace(-1.0, 1.0, p.n_steps * p.n_det * 3, device="cuda").reshape(1, p.n_steps, p.n_det, 3)
            ids.append(b.submit(p, [f[3]], obs=obs))
        done = b.run_to_completion(chunk=64)
        torch.cuda.synchronize()
        by_id = {r["id"]: r for r in done}
        got.append([by_id[i][k].clone() for i in ids for k in ("traces", "g_eps", "g_sigma")])
        b.close()
        for p in ps:
            p.close()
    for a, b in zip(*got):
        assert torch.isfinite(a).all() and torch.equal(_bits(torch, a), _bits(torch, b))

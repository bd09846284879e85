"""What a batched job is charged: the bytes of its problem without the plans of resident solves, which a batch never
builds.  The values are those that dd_footprint_bytes gave before there were such plans, and the fields' pads."""

import ctypes
import math

import pytest

import synth

PADS = 64          # four floats past each of the four levels
CASES = [          # n_outer, fem_cells, n_steps, ckpt_every, detector faces, sources, bytes
    ((25, 25, 25), (8, 8, 8), 300, 300, 63, 1, 5203520),
    ((64, 64, 64), (32, 32, 32), 400, 64, 1, 2, 213180160),
    ((37, 35, 41), (12, 10, 14), 120, 32, 37, 3, 12917440),
    ((96, 96, 96), (48, 48, 48), 600, 64, 1, 1, 598229280),
    ((160, 160, 160), (64, 64, 64), 100, 25, 1, 1, 872803816),
]


def _desc(n, cells, nt, ck, det):
    lo = tuple((a - b) // 2 for a, b in zip(n, cells))
    return synth.ProblemDesc(n_outer=n, h=0.05, origin=(0.0, 0.0, 0.0), fem_lo=lo, fem_cells=cells,
                             dt=0.5 * 0.05 / math.sqrt(3.0), n_steps=nt, ckpt_every=ck, detector_faces=det,
                             absorbing_faces=3)


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])))
def test_batched_job_is_charged_no_plans(case):
    from paper_2508_07780_amd import Problem, serving
    d = _desc(*case[:5])
    assert Problem.footprint_bytes(d, case[5], batched=True) == case[6] + PADS
    plans = Problem.footprint_bytes(d, case[5]) - case[6] - PADS
    assert (plans > 0) == (case[0][0] < 100)

    class Request:
        workload = type("W", (), {"desc": d, "sources": [None] * case[5]})
    assert serving.job_footprint(Request, alone=True) - serving.job_footprint(Request) == plans


def test_invalid_descriptor_is_0():
    from paper_2508_07780_amd import _lib
    lib = _lib.load()
    c = _lib.make_desc(_desc(*CASES[0][:5]))
    assert lib.dd_batch_footprint_bytes(ctypes.byref(c), -1) == 0
    c.n_steps = 0
    assert lib.dd_batch_footprint_bytes(ctypes.byref(c), 1) == lib.dd_footprint_bytes(ctypes.byref(c), 1) == 0


@pytest.mark.gpu
def test_batched_job_stays_within_its_charge():
    import torch
    from paper_2508_07780_amd import DDError, Problem
    from paper_2508_07780_amd.batch import Batch
    w = synth.small("tiny")
    charge = Problem.footprint_bytes(w.desc, 1, batched=True)
    ps = [Problem(w.desc) for _ in range(3)]
    for p in ps:
        p.set_coefficients(torch.tensor(w.eps, dtype=torch.float32, device="cuda"),
                           torch.tensor(w.sigma, dtype=torch.float32, device="cuda"))
    obs = torch.zeros((1, w.desc.n_steps, ps[0].n_det, 3), dtype=torch.float32, device="cuda")
    b = Batch(4, hbm_budget=2 * charge)
    b.submit(ps[0], w.sources, obs=obs)
    b.submit(ps[1], w.sources, obs=obs)                # room for exactly two
    with pytest.raises(DDError):
        b.submit(ps[2], w.sources, obs=obs)
    assert len(b.run_to_completion(chunk=64)) == 2
    assert all(p.device_bytes() <= charge for p in ps)
    b.close()
    for p in ps:
        p.close()


@pytest.mark.gpu
def test_plans_of_its_own_solves_are_charged(monkeypatch):
    import torch
    from paper_2508_07780_amd import DDError, Problem
    from paper_2508_07780_amd.batch import Batch
    monkeypatch.setenv("DD_RESIDENT", "1")
    w = synth.small("tiny")
    charge = Problem.footprint_bytes(w.desc, 1, batched=True)
    p = Problem(w.desc)
    p.set_coefficients(torch.tensor(w.eps, dtype=torch.float32, device="cuda"),
                       torch.tensor(w.sigma, dtype=torch.float32, device="cuda"))
    p.forward(w.sources, save=True)
    assert p.resident_stats("forward")["blocks"] > 0
    obs = torch.zeros((1, w.desc.n_steps, p.n_det, 3), dtype=torch.float32, device="cuda")
    small, large = Batch(1, hbm_budget=charge), Batch(1, hbm_budget=Problem.footprint_bytes(w.desc, 1))
    with pytest.raises(DDError):
        small.submit(p, w.sources, obs=obs)
    large.submit(p, w.sources, obs=obs)
    assert len(large.run_to_completion(chunk=64)) == 1
    small.close()
    large.close()
    p.close()

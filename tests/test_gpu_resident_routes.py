"""Which kernel takes a resident solve, and that each of them equals the launches bit for bit.

* every variant of the resident kernels takes its solves itself, and equals the launches;
* a called-off launch's solves are taken by the fallback kernel, at a rate near the launches';
* launches of unequal sizes on several streams are not called off;
* solves beside work that fills the GPU;
* a solve whose launch is called off, with the streaming variant of the launches forced
  (DD_FD_NT=1): the kernel that takes it lays out its own blocks.
"""

import math

import pytest

from tests.resident_forms import VARIANTS, problem, variant
from tests.test_gpu_resident import FORMS, _form, _problem, _run, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["minimal", "one_over", "sides"])
def test_called_off_with_streaming_launches(name, monkeypatch):
    import torch
    form = _form(name)
    monkeypatch.setenv("DD_FD_NT", "1")
    got = []
    for mode in (0, 2):
        print(f"[gpu] {name} DD_FD_NT=1 DD_RESIDENT={mode}", flush=True)
        p = _problem(torch, monkeypatch, form, mode)
        got.append(_run(torch, p, form[3][:1]))
        p.close()
    assert all(_same(torch, *got)), _same(torch, *got)


def _solves(n_src):
    """Forward and adjoint solves of a _run of n_src sources."""
    return {"forward": 3 * n_src, "adjoint": 4 * n_src}


@pytest.mark.parametrize("name", sorted(VARIANTS))
def test_variants_equal_launches_bit_for_bit(name, monkeypatch):
    import torch
    form = problem(name)
    got = []
    for mode in (0, 1):
        print(f"[gpu] {name} DD_RESIDENT={mode}", flush=True)
        p = _problem(torch, monkeypatch, form, mode)
        got.append(_run(torch, p, form[3]))
        assert float(got[-1][0].abs().max()) > 0
        for i, which in enumerate(("forward", "adjoint")):
            s = p.resident_stats(which)
            assert s["called_off"] == s["fallback"] == 0
            assert s["solves"] == (_solves(2)[which] if mode else 0)
            if mode:
                assert variant(s["run"], s["fem_nodes"]) == VARIANTS[name][7 + i], s
        p.close()
    assert all(_same(torch, *got)), _same(torch, *got)


@pytest.mark.parametrize("name", sorted(FORMS))
def test_solves_run_resident(name, monkeypatch):
    import torch
    form = _form(name)
    p = _problem(torch, monkeypatch, form, 1)
    _run(torch, p, form[3])
    for which in ("forward", "adjoint"):
        s = p.resident_stats(which)
        assert (s["solves"], s["called_off"], s["fallback"]) == (_solves(2)[which], 0, 0), (which, s)
    p.close()


@pytest.mark.parametrize("name", ["minimal", "one_over"])
def test_called_off_solves_are_taken(name, monkeypatch):
    import torch
    form = _form(name)
    p = _problem(torch, monkeypatch, form, 2)
    _run(torch, p, form[3][:1])
    for which in ("forward", "adjoint"):
        s = p.resident_stats(which)
        assert s["solves"] == 0 and s["fallback"] == _solves(1)[which] and s["called_off"] >= s["fallback"], (which, s)
    p.close()


def test_unequal_launches_on_three_streams(monkeypatch):
    """One launch that fills the GPU for a while and two small ones that fit beside each other, not beside it."""
    import copy
    import torch
    long = copy.deepcopy(problem("f4"))
    long[0].n_steps = 60000
    long[0].ckpt_every = 60000
    forms = [long, _form("one_over"), _form("one_over")]
    ps = [_problem(torch, monkeypatch, f, 1) for f in forms]
    want = ps[1].forward(forms[1][3][:1], save=False).clone()
    ps[2].forward(forms[2][3][:1], save=False)
    out = [torch.empty((1, p.n_steps, p.n_det, 3), dtype=torch.float32, device="cuda") for p in ps]
    streams = [torch.cuda.Stream() for _ in ps]
    torch.cuda.synchronize()
    for p, f, o, s in zip(ps, forms, out, streams):
        with torch.cuda.stream(s):
            p.forward(f[3][:1], save=False, out=o)
    torch.cuda.synchronize()
    stats = [p.resident_stats("forward") for p in ps]
    print("[gpu]", stats, flush=True)
    assert stats[0]["blocks"] > 256 - stats[1]["blocks"] and 2 * stats[1]["blocks"] <= 256
    assert [s["called_off"] for s in stats] == [0, 0, 0]
    assert torch.equal(out[1], want) and torch.equal(out[2], want)
    for p in ps:
        p.close()


def test_called_off_solves_keep_their_rate(monkeypatch):
    """A solve whose launch was called off takes a few times as long as by launches (5 measured), not hundreds."""
    import time
    import torch
    form = problem("cube64")
    form[0].n_steps = form[0].ckpt_every = 200
    took = []
    for mode in (0, 2):
        p = _problem(torch, monkeypatch, form, mode)
        tr = p.forward(form[3][1:], save=True).clone()
        best = math.inf
        for _ in range(3):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            p.forward(form[3][1:], save=True, out=tr)
            p.adjoint(tr)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        if mode:
            assert p.resident_stats("forward")["fallback"] == p.resident_stats("adjoint")["fallback"] + 1 == 4
        took.append(best)
        p.close()
    print(f"[gpu] {took[0] * 1e3:.2f} ms by launches, {took[1] * 1e3:.2f} ms called off", flush=True)
    assert took[1] <= 30 * took[0]


def test_launches_for_a_while_after_a_call_off(monkeypatch):
    """A problem whose launch was called off runs its next 16 solves by launches, then tries again, and pauses for 32."""
    import torch
    form = _form("minimal")
    ref = _problem(torch, monkeypatch, form, 0)
    want = ref.forward(form[3], save=True).clone()
    p = _problem(torch, monkeypatch, form, 3)
    tries = []
    for _ in range(30):                              # two solves each
        before = p.resident_stats("forward")
        out = p.forward(form[3], save=True)
        torch.cuda.synchronize()
        after = p.resident_stats("forward")
        assert torch.equal(out, want)
        tries.append((after["called_off"] - before["called_off"], after["fallback"] - before["fallback"]))
    # the second solve of a call that was called off does not wait again
    assert tries[0] == tries[9] == tries[26] == (1, 2)
    assert sum(t != (0, 0) for t in tries) == 3
    p.close()
    ref.close()


def test_beside_work_that_fills_the_gpu(monkeypatch):
    """Solves on one stream while large products keep the GPU full on another: whichever kernel takes a solve, its results
    are the launches'."""
    import torch
    form = problem("cube64")
    form[0].n_steps = form[0].ckpt_every = 60
    ref = _problem(torch, monkeypatch, form, 0)
    want = _run(torch, ref, form[3])
    ref.close()
    p = _problem(torch, monkeypatch, form, 1)
    a = torch.randn((8192, 8192), device="cuda")
    c = torch.empty_like(a)
    other, mine = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(other):
        for _ in range(40):
            torch.mm(a, a, out=c)
        end = torch.cuda.Event()
        end.record()
    with torch.cuda.stream(mine):
        for _ in range(4):
            got = _run(torch, p, form[3])
            assert all(_same(torch, got, want)), _same(torch, got, want)
        stats = [p.resident_stats(w) for w in ("forward", "adjoint")]
    print(f"[gpu] {stats}", flush=True)
    for s, n in zip(stats, (_solves(2)["forward"], _solves(2)["adjoint"])):
        assert s["solves"] + s["fallback"] <= 4 * n and s["called_off"] <= s["fallback"]
    p.close()

"""Building the plan of resident solves inside a call: it does not wait for the caller's stream, leaves another thread's
capture alone, and without memory for the plan the solves go on by launches and nothing is held."""

import threading

import pytest

from tests.test_gpu_resident import _form, _problem

pytestmark = pytest.mark.gpu


def test_does_not_wait_for_the_stream(monkeypatch):
    import torch
    form = _form("one_over")
    ps = [_problem(torch, monkeypatch, form, m) for m in (0, 1, 1)]
    want = ps[0].forward(form[3][:1], save=False).clone()
    ps[1].forward(form[3][:1], save=False)               # the kernels' first use
    out = torch.empty_like(want)
    st = torch.cuda.Stream()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    torch.cuda._sleep(10 ** 7)
    b.record()
    torch.cuda.synchronize()
    cycles = int(10 ** 7 * 1000.0 / a.elapsed_time(b))   # about a second
    with torch.cuda.stream(st):
        torch.cuda._sleep(cycles)
        slept = torch.cuda.Event()
        slept.record()
        ps[2].forward(form[3][:1], save=False, out=out)
        assert not slept.query()
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    assert ps[2].resident_stats("forward")["solves"] == 1
    for p in ps:
        p.close()


def test_beside_a_capture_of_another_thread(monkeypatch):
    import torch
    form = _form("one_over")
    ps = [_problem(torch, monkeypatch, form, m, allocator=None) for m in (0, 1)]
    want = ps[0].forward(form[3][:1], save=False).clone()
    out = torch.empty_like(want)
    st = torch.cuda.Stream()
    errors = []

    def work():
        try:
            with torch.cuda.stream(st):
                ps[1].forward(form[3][:1], save=False, out=out)
        except BaseException as e:  # noqa: BLE001
            errors.append(e)

    x = torch.ones(1000, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="global"):
        y = x * 2
        t = threading.Thread(target=work)
        t.start()
        t.join()
        y += 1
    assert not errors, errors
    torch.cuda.synchronize()
    assert torch.equal(out, want) and ps[1].resident_stats("forward")["solves"] == 1
    for _ in range(3):
        x += 1
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, 2 * x + 1)
    for p in ps:
        p.close()


@pytest.mark.parametrize("granted", [0, 1, 2])
def test_without_memory_for_the_plan(granted, monkeypatch):
    import torch
    from paper_2508_07780_amd import solver
    form = _form("one_over")
    ref = _problem(torch, monkeypatch, form, 0)
    want = ref.forward(form[3], save=False).clone()
    ref.close()
    left = [None]                       # allocations still granted (None: all)
    alloc = solver.TorchAllocator._alloc

    def some(self, nbytes, ctx):
        if left[0] is not None:
            if not left[0]:
                return None
            left[0] -= 1
        return alloc(self, nbytes, ctx)

    monkeypatch.setattr(solver.TorchAllocator, "_alloc", some)
    p = _problem(torch, monkeypatch, form, 1)
    held = p.device_bytes()
    left[0] = granted
    out = p.forward(form[3], save=False)
    left[0] = None
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    stats = p.resident_stats("forward")
    print(f"[gpu] granted {granted}: {stats}, {p.device_bytes() - held} bytes more", flush=True)
    assert (stats["blocks"] > 0) == (p.device_bytes() > held)
    assert stats["solves"] == (2 if stats["blocks"] else 0)
    p.close()

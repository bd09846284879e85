"""Which kernel takes a resident solve, and that each of them equals the launches bit for bit.

* every variant of the resident kernels takes its solves itself, and equals the launches;
* a called-off launch's solves are taken by the fallback kernel;
* a solve whose launch is called off, with the streaming variant of the launches forced
  (DD_FD_NT=1): the kernel that takes it lays out its own blocks.
"""

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

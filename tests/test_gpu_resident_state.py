"""The field state that a resident solve leaves for the calls after it."""

import pytest

from tests.test_gpu_resident import _form, _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
def test_finite_after_a_diverged_start(mode, monkeypatch):
    """Initial data whose level before the start overflows inside the box: that solve diverges, the next one from rest does
    not, by launches or resident."""
    import torch
    from paper_2508_07780_amd import DDError
    form = _form("one_over")
    d = form[0]
    p = _problem(torch, monkeypatch, form, mode)
    p.forward(form[3][:1], save=False)
    p.check_finite()
    f0 = torch.zeros((p.n_grid, 3), dtype=torch.float32, device="cuda")
    f1 = torch.zeros_like(f0)
    x, y, z = (a + n // 2 for a, n in zip(d.fem_lo, d.fem_cells))
    node = x + d.n_outer[0] * (y + d.n_outer[1] * z)
    f0[node], f1[node] = 3.4e38, -3.0e38
    p.set_initial_data(f0, f1)
    p.forward(form[3][:1], save=False)
    with pytest.raises(DDError):
        p.check_finite()
    p.set_initial_data(None, None)
    p.forward(form[3][:1], save=False)
    assert p.resident_stats("forward")["solves"] == 2 * mode
    p.check_finite()
    p.close()


@pytest.mark.parametrize("mode", [0, 1])
def test_non_finite_fields_are_found(mode, monkeypatch):
    import torch
    from paper_2508_07780_amd import DDError
    form = _form("one_over")
    p = _problem(torch, monkeypatch, form, mode)
    tr = p.forward(form[3][:1], save=True)
    p.check_finite()
    cot = torch.zeros_like(tr)
    cot[0, -2, 7, 1] = float("nan")
    p.adjoint(cot)
    with pytest.raises(DDError):
        p.check_finite()
    p.close()

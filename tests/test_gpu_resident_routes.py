"""Which kernel takes a resident solve, and that each of them equals the launches bit for bit.

* a solve whose launch is called off, with the streaming variant of the launches forced
  (DD_FD_NT=1): the kernel that takes it lays out its own blocks.
"""

import pytest

from tests.test_gpu_resident import _form, _problem, _run, _same

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

"""The lattice blocks a caller mesh's nodes are grouped by (8x4x4 on boxes of few blocks, else 8^3).

The default on a small box is the quarter block, bit for bit; against 8^3 the elements of a node are
summed in another order: FP32 rounding, a few 1e-7 per step of some hundred sums that the leapfrog
carries on without growth, so 1e-5 of the norm holds with a wide margin.
"""

import numpy as np
import pytest

import synth
from tests.test_gpu_mesh import _refined

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["ragged", "skinlet"])
def test_blocks_agree(name, monkeypatch):
    import torch
    from paper_2508_07780_amd import Problem
    out = {}
    w, _, mesh, eps, sig = _refined(name, {"ragged": 0.6, "skinlet": 0.3}[name])
    for pb in (None, "8,4,4", "8,8,8"):
        if pb:
            monkeypatch.setenv("DD_FEM_PB", pb)
        print(f"[gpu] {name} blocks {pb}", flush=True)
        p = Problem(w.desc, mesh=mesh)
        p.set_coefficients(torch.tensor(np.asarray(eps), dtype=torch.float32, device="cuda"),
                           torch.tensor(np.asarray(sig), dtype=torch.float32, device="cuda"))
        tr = p.forward(w.sources, save=True).clone()
        p.adjoint((0.3 * tr).contiguous())
        out[pb] = [tr] + [g.clone() for g in p.gradient()]
        torch.cuda.synchronize()
        p.close()
    for a, b in zip(out[None], out["8,4,4"]):
        assert torch.equal(a, b)
    for a, b in zip(out[None], out["8,8,8"]):
        assert float((a.double() - b.double()).norm() / b.double().norm()) <= 1e-5

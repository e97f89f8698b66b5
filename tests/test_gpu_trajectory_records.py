"""Trajectory gradients with the stage records kept by the forward pass: against
the same gradients with every record recomputed from its checkpoint, for no, some
and all segments kept, and for a second backward pass through one graph.

Recorded and plain steps run one kernel on one plan with the same operands in the
same order, so paths and gradients may differ only where the two round differently:
bounds of a few units of float32 rounding (2^-24) per step, against the largest
entry."""
import pytest
import torch

import llg_inputs as li

pytestmark = pytest.mark.gpu

C_PY = 0.29
N_SEG, SEG = 4, 5
TOL = 4 * 2.0 ** -24 * N_SEG * SEG


def gradients(disk, m0, noise, kept, monkeypatch, again=False):
    from paper_1207_2192_amd import LLGParams, adjoint
    monkeypatch.setattr(adjoint, "_kept_segments", lambda n, floats, device: min(n, kept))
    prm = LLGParams(alpha=0.02, c=C_PY, dtau=0.03, temp=0.0 if noise is None else 0.01, renorm=noise is not None)
    m = m0.clone().requires_grad_(True)
    a = torch.tensor(0.02, dtype=torch.float64, requires_grad=True)
    c = torch.tensor(C_PY, dtype=torch.float64, requires_grad=True)
    rc = adjoint.core_trajectory(m, a, c, disk, prm, N_SEG, SEG, 5.0, noise)
    loss = ((rc - torch.ones_like(rc)) ** 2).sum()
    first = torch.autograd.grad(loss, (m, a, c), retain_graph=again)
    out = [first] + ([torch.autograd.grad(loss, (m, a, c))] if again else [])
    disk.check()
    return rc.detach(), out


def same(x, y):
    assert float((x - y).abs().max()) <= TOL * max(float(y.abs().max()), 1e-30)


@pytest.mark.parametrize("noise", [None, (5, 700, 1)])
@pytest.mark.parametrize("R", [30.0, 80.0])
def test_kept_and_recomputed_records_give_one_gradient(R, noise, monkeypatch):
    from paper_1207_2192_amd import Disk
    disk = Disk.build(R, 10.0)
    m0 = torch.from_numpy(li.vortex_ansatz(disk.D[0], 2.6, 0.4)).float().cuda().reshape(-1)
    rc0, (g0,) = gradients(disk, m0, noise, 0, monkeypatch)
    for kept in (2, N_SEG):
        rc, passes = gradients(disk, m0, noise, kept, monkeypatch, again=True)
        same(rc, rc0)
        for g in passes:
            for x, y in zip(g, g0):
                same(x, y)


def test_no_record_without_a_gradient(monkeypatch):
    from paper_1207_2192_amd import Disk, LLGParams, adjoint
    disk = Disk.build(30.0, 10.0)
    m = torch.from_numpy(li.vortex_ansatz(disk.D[0], 2.6, 0.4)).float().cuda().reshape(-1).requires_grad_(True)
    monkeypatch.setattr(adjoint, "_record", lambda *a: pytest.fail("recorded without a backward pass"))
    with torch.no_grad():
        rc = adjoint.core_trajectory(m, 0.02, C_PY, disk, LLGParams(alpha=0.02, c=C_PY, dtau=0.03), 2, 3, 5.0)
    assert rc.shape == (3, 2) and not rc.requires_grad

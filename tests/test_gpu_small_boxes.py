"""Relaxation and RK4 adjoint where their row tiles are mostly padding: boxes from the
smallest to the whole of P = 64 and 128, under plans of both radices and several unit
groups, one workgroup and many, against the float64 oracle.

Tolerances.  Relaxation: a sweep sums about 30 float32 terms of size 1 to 8 per
component and divides by their norm, 32 units of rounding (2^-24) a sweep, and sweeps
contract: 5 x 32 x 2^-24.  Adjoint: 1e-5 of the largest entry, as for larger disks."""
import numpy as np
import pytest
import torch

import llg_inputs as li
import oracle
from oracle.dynamics import rk4_step as o_rk4
from oracle.relax import relax as o_relax

pytestmark = pytest.mark.gpu
C_PY = 0.14298555
PLANS = [(1, 0), (1, 1), (2, 3), (4, 1)]
BOXES = [2, 5, 24, 32, 33, 48, 64]


def dev(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda").reshape(-1).contiguous()


def plans(disk):
    for ug, pol in PLANS:
        for wg in ([1], [3], None):
            disk.tune(ug, wg, pol)
            print(disk.D[0], ug, pol, disk.workgroups, flush=True)
            yield


@pytest.mark.parametrize("D", BOXES)
def test_relaxation(D):
    from paper_1207_2192_amd import Disk, LLGParams
    disk, od = Disk.build(float(D), 6.0), oracle.Disk(float(D), 6.0)
    assert disk.D[0] == D
    m0 = dev(li.smooth_random_field(D, 4))
    ref = o_relax(m0.view(3, D, D).double().cpu(), od, oracle.Params(c=C_PY), (0.6, -0.4), tol=1e-30,
                  max_sweeps=5)[0]
    for _ in plans(disk):
        m = m0.clone()
        out = disk.relax(m, [(0.6, -0.4)], LLGParams(c=C_PY), tol=1e-30, max_sweeps=5)
        disk.check()
        assert float(out[0, 2]) == 5
        assert float((m.view(3, D, D).double().cpu() - ref).abs().max()) <= 5 * 32 * 2.0 ** -24


@pytest.mark.parametrize("D", BOXES)
def test_rk4_adjoint(D):
    from paper_1207_2192_amd import Disk, LLGParams
    disk, od = Disk.build(float(D), 6.0), oracle.Disk(float(D), 6.0)
    kw = dict(dtau=0.05, hext=(0.02, -0.01, 0.03))
    p = LLGParams(alpha=0.07, c=C_PY, **kw)
    m0, yb = dev(li.smooth_random_field(D, 4)), dev(li.random_unit_field(D, 9) * od.mask.numpy())
    mr = m0.view(3, D, D).double().cpu().requires_grad_(True)
    a, c = (torch.tensor(v, dtype=torch.float64, requires_grad=True) for v in (0.07, C_PY))
    y = o_rk4(mr, od, oracle.Params(alpha=a, c=c, **kw), 2)
    gm, ga, gc = torch.autograd.grad((y * yb.view(3, D, D).double().cpu() * od.mask).sum(), (mr, a, c))
    gm = od.apply_mask(gm)
    for _ in plans(disk):
        rec = torch.empty(16 * disk.state_size, dtype=torch.float32, device="cuda")
        disk.rk4_record(m0.clone(), 2, p, rec)
        got, pg = yb.clone(), torch.zeros(2, dtype=torch.float64, device="cuda")
        disk.rk4_vjp(rec, 2, got, pg, p)
        disk.check()
        assert float((got.view(3, D, D).double().cpu() - gm).abs().max()) <= 1e-5 * float(gm.abs().max())
        for x, r in zip(pg.tolist(), (float(ga), float(gc))):
            assert abs(x - r) <= 1e-5 * abs(r) + 1e-6

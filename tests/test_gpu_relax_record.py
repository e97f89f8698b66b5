"""The record of a relaxation (multipliers, residual, constraint), whose partial sums
every workgroup of a disk reduces for itself: one to 129 workgroups, so that the
lanes that take eight workgroups each go round once and twice, with and without a
remainder.

After one sweep the states are equal bit for bit and the sums differ in their order
alone: terms of m_z^2 dx add up to less than 1e3, at 1e4 roundings of 1e-16 1e-9 at
worst and 1e-13 in practice; multipliers are their quotients by sums of order 100.
1e-11.  Twenty sweeps against the float64 oracle: 32 units of float32 rounding a
sweep in the state; in the multipliers 1e-4, that error of about 50 core cells at ten
cells from the target over a Jacobian of order 100."""
import pytest
import torch

import llg_inputs as li
import oracle
from oracle.relax import relax as o_relax

pytestmark = pytest.mark.gpu
C_PY = 0.14298555
X = [(4.0, 0.0), (0.0, -2.0)]
COUNTS = ([1, 1], [3, 8], [16, 9], [17, 16], [33, 63], [64, 65], [66, 72], [129, 129])


def start(disk):
    return disk.pack([torch.tensor(li.vortex_ansatz(D, 3.0, -2.0), dtype=torch.float32, device="cuda").reshape(-1)
                      for D in disk.D])


@pytest.mark.parametrize("cut", [0.0, 21.0])
def test_one_sweep_has_one_record(cut):
    from paper_1207_2192_amd import Disk, LLGParams
    disk = Disk.batch([100.0, 70.0], [20.0, 9.0])
    m0, ref = start(disk), None
    for wg in COUNTS:
        disk.tune(1, wg, 0)
        assert disk.workgroups == wg
        m = m0.clone()
        out = disk.relax(m, X, LLGParams(c=C_PY), max_sweeps=1, cutoff_nm=cut)
        disk.check()
        print(wg, out[:, :6].tolist(), flush=True)
        ref = (m, out) if ref is None else ref
        assert torch.equal(m, ref[0])
        assert torch.equal(out[:, 2:4], ref[1][:, 2:4])               # sweeps; the largest residual is one cell's
        assert float((out - ref[1]).abs().max()) <= 1e-11
    assert float(ref[1][:, :2].abs().max()) > 1e-4                     # multipliers that could differ


@pytest.mark.parametrize("wg", [1, 47, 129])
def test_twenty_sweeps_follow_the_oracle(wg):
    from paper_1207_2192_amd import Disk, LLGParams
    disk, od = Disk.build(100.0, 20.0), oracle.Disk(100.0, 20.0)
    disk.tune(1, [wg], 0)
    assert disk.workgroups == [wg]
    m = start(disk)
    mo, lam, sweeps, res, C = o_relax(m.view(3, 100, 100).double().cpu(), od, oracle.Params(c=C_PY), X[0], tol=1e-30,
                                      max_sweeps=20, cutoff_nm=21.0)
    out = disk.relax(m, X[:1], LLGParams(c=C_PY), tol=1e-30, max_sweeps=20, cutoff_nm=21.0).cpu()[0]
    disk.check()
    print(wg, out.tolist(), lam.tolist(), res, C.tolist(), flush=True)
    assert int(out[2]) == sweeps == 20
    assert float((m.view(3, 100, 100).double().cpu() - mo).abs().max()) <= 20 * 32 * 2.0 ** -24
    assert float((out[:2] - lam).abs().max()) <= 1e-4
    assert abs(float(out[3]) - res) <= 20 * 32 * 2.0 ** -24 * 10 and float((out[4:6] - C).abs().max()) <= 1e-2

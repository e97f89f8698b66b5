"""The library's own plan gives few large disks two unit groups a workgroup; what
that must not change: explicit workgroup counts at creation, and an on-chip limit
on a handle whose plan nobody chose."""
import pytest
import torch

import llg_inputs as li

pytestmark = pytest.mark.gpu


def steps(disk):
    from paper_1207_2192_amd import LLGParams
    m = disk.pack([torch.tensor(li.vortex_ansatz(D, 1.4, -0.7), dtype=torch.float32, device="cuda").reshape(-1)
                   for D in disk.D])
    disk.rk4_step(m, 4, LLGParams(alpha=0.02, c=0.14298555, dtau=0.03))
    disk.check()
    return m


@pytest.mark.parametrize("boxes,counts", [([100.0], [120]), ([100.0, 130.0], [70, 200]), ([100.0, 30.0], [9, 3])])
def test_explicit_counts_are_kept(boxes, counts):
    from paper_1207_2192_amd import Disk
    disk = Disk.batch(boxes, [20.0] * len(boxes), wg_per_disk=counts)
    print(disk.workgroups, disk.launch_shape(), flush=True)
    assert disk.workgroups == counts and disk.launch_shape()[0] == 1
    assert torch.equal(steps(disk), steps(Disk.batch(boxes, [20.0] * len(boxes), wg_per_disk=[2] * len(boxes))))


def test_on_chip_limit_on_a_default_plan():
    from paper_1207_2192_amd import Disk
    disk = Disk.build(100.0, 20.0)
    ref = steps(disk)
    for limit in (64, 128, 0):
        disk.set_on_chip(limit)
        assert disk.on_chip == limit
        assert torch.equal(steps(disk), ref)
    disk.set_on_chip(64)
    with pytest.raises(Exception, match="one unit group"):
        disk.tune(2)
    disk.set_on_chip(0)
    disk.tune(2)
    with pytest.raises(Exception, match="one unit group"):       # two by the caller's choice
        disk.set_on_chip(64)
    assert disk.on_chip == 0 and disk.launch_shape()[0] == 2
    assert torch.equal(steps(disk), ref)

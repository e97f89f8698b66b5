"""Plans for every mode: one workgroup of several unit groups per CU.  Workgroup
counts around what one XCD's 32 CUs hold, next to a second disk; each transform is
computed the same way whichever workgroup carries it, so states are equal bit for
bit, and a plan never counts on more workgroups than CUs."""
import pytest
import torch

import llg_inputs as li

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ug", [2, 4])
def test_plans_of_several_unit_groups_stay_within_the_cus(ug):
    from paper_1207_2192_amd import Disk, LLGParams
    disk = Disk.batch([100.0, 60.0], [20.0, 10.0])
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    m0 = disk.pack([torch.tensor(li.vortex_ansatz(D, 2.0, -1.0), dtype=torch.float32, device="cuda").reshape(-1)
                    for D in disk.D])
    p = [LLGParams(alpha=0.02, c=0.14298555, dtau=0.04)] * disk.n
    ref = None
    for wg in ([31, 9], [32, 8], [33, 17], None):
        disk.tune(ug, wg, 0)
        print(ug, wg, disk.workgroups, disk.launch_shape(), flush=True)
        assert sum(disk.workgroups) <= cus
        m = m0.clone()
        disk.rk4_step(m, 3, p)
        disk.check()
        ref = m if ref is None else ref
        assert torch.equal(m, ref)

"""Group barrier of a disk on few workgroups (one counter) and on many (a
counter per line): around the switch at 16 workgroups, at counts that leave the
lines unequal, and at the largest.  Every transform is computed the same way
whichever workgroup carries it, so all counts give the same bits; the step that
every stage waits at the barrier makes a lost arrival a timeout."""
import pytest
import torch

import llg_inputs as li

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["rk4", "heun_series", "relax"])
def test_workgroup_counts_around_the_counter_switch(kind):
    from paper_1207_2192_amd import Disk, LLGParams
    disk = Disk.batch([100.0, 70.0], [20.0, 9.0])
    m0 = disk.pack([torch.tensor(li.vortex_ansatz(D, 3.0, -2.0), dtype=torch.float32, device="cuda").reshape(-1)
                    for D in disk.D])
    p = LLGParams(alpha=0.05, c=0.14298555, dtau=0.04, temp=0.01 if kind == "heun_series" else 0.0,
                  renorm=kind == "heun_series")
    ref = None
    for wg in ([16, 15], [17, 16], [18, 33], [31, 47], [64, 32], [129, 129]):
        disk.tune(1, wg, 0)
        print(kind, disk.workgroups, flush=True)
        m = m0.clone()
        if kind == "rk4":
            disk.rk4_step(m, 12, p)
        elif kind == "heun_series":
            disk.heun_series(m, 12, p, 5, seed=3, step0=0)
        else:
            disk.relax(m, [(4.0, 0.0), (0.0, 2.0)], p, max_sweeps=1)   # one sweep: no float64 sums feed back
        disk.check()
        ref = m if ref is None else ref
        assert torch.equal(m, ref), wg

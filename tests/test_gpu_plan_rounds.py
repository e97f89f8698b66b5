"""Plans that step a batch in several launches one after the other: an odd number
of disks of mixed boxes, so that the launches differ in their workgroup maps, through
every call that a persistent launch serves and through graphs.  Each transform is
computed the same way whichever workgroup and launch carries it, so states equal
those of one launch bit for bit; float64 sums follow the plan's workgroups, equal to
1e-12 of their size."""
import pytest
import torch

import llg_inputs as li

pytestmark = pytest.mark.gpu
C_PY = 0.14298555
BOXES = [100, 30, 130, 48, 66, 20, 101]


def close(a, b):
    return float((a - b).abs().max()) <= 1e-12 * float(b.abs().max())


@pytest.mark.parametrize("ug,pol", [(1, 0), (1, 3), (4, 3)])
def test_rounds_equal_a_single_launch(ug, pol):
    from paper_1207_2192_amd import Disk, LLGParams
    disk = Disk.batch([float(D) for D in BOXES], [0.1 * D for D in BOXES])
    m0 = disk.pack([torch.tensor(li.vortex_ansatz(D, 1.4, -0.7), dtype=torch.float32, device="cuda").reshape(-1)
                    for D in disk.D])
    p = [LLGParams(alpha=0.02, c=C_PY, dtau=0.03)] * disk.n
    ph = [LLGParams(alpha=0.1, c=C_PY, dtau=0.02, temp=0.008, renorm=True)] * disk.n
    X = [(2.0, 0.0)] * disk.n

    def run(rounds):
        assert disk.debug_rounds(ug, pol, rounds) == rounds == disk.debug_rounds()
        print(ug, pol, "rounds", rounds, disk.launch_shape(), disk.workgroups, flush=True)
        out = {k: m0.clone() for k in ("rk4", "heun", "rk4 series", "heun series", "relax", "record", "vjp", "graph")}
        disk.rk4_step(out["rk4"], 6, p)
        disk.set_step(11)
        disk.heun_step(out["heun"], 6, ph, seed=5, step0=None, replica=3)
        assert disk.get_step() == 17
        sums = [disk.rk4_series(out["rk4 series"], 6, p, 2),
                disk.heun_series(out["heun series"], 6, ph, 4, seed=5, step0=11, replica=3)]
        disk.relax(out["relax"], X, p, max_sweeps=1)               # one sweep: no float64 sums feed back
        rec = torch.empty(8 * 2 * disk.state_size, dtype=torch.float32, device="cuda")
        disk.rk4_record(out["record"], 2, p, rec)
        grad = torch.zeros(2 * disk.n, dtype=torch.float64, device="cuda")
        disk.rk4_vjp(rec, 2, out["vjp"], grad, p)
        sums.append(grad)
        disk.set_step(11)
        g = disk.graph("heun", out["graph"], 2, ph, seed=5, replica=3)
        for _ in range(3):
            g.launch()
            float(torch.randn(1 << 16, device="cuda").sum())
        disk.check()
        assert disk.get_step() == 17
        g.close()
        assert torch.equal(out["graph"], out["heun"])
        return out, sums

    ref, ref_sums = run(1)
    for rounds in (2, 3):
        got, sums = run(rounds)
        for k in ref:
            assert torch.equal(got[k], ref[k]), k
        assert all(close(a, b) for a, b in zip(sums, ref_sums))
    for bad in (-1, disk.n + 1):
        with pytest.raises(Exception, match="rounds"):
            disk.debug_rounds(1, 0, bad)


def test_graph_of_two_launches_follows_eager_rk4():
    from paper_1207_2192_amd import Disk, LLGParams
    disk = Disk.batch([66.0, 40.0, 100.0], [10.0, 8.0, 20.0])
    p = [LLGParams(alpha=0.02, c=C_PY, dtau=0.03)] * disk.n
    mg = disk.pack([torch.tensor(li.vortex_ansatz(D, 1.4, -0.7), dtype=torch.float32, device="cuda").reshape(-1)
                    for D in disk.D])
    me = mg.clone()
    assert disk.debug_rounds(1, 0, 2) == 2
    g = disk.graph("rk4", mg, 5, p)
    disk.tune(2)                                   # the graph keeps its plan
    assert disk.debug_rounds() == 1
    for rep in range(4):
        g.launch()
        float(torch.randn(1 << 16, device="cuda").sum())
        disk.debug_rounds(1, 0, 1 + rep % 2)
        disk.rk4_step(me, 5, p)
        disk.check()
        assert torch.equal(mg, me), rep
    g.close()
